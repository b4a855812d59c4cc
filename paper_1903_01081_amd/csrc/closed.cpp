// Closed-form solve of a component: sizes, lists for its numeric kernel and
// the row programs of the step kernels (see closed.h). No HIP calls.
#include "closed.h"

#include <algorithm>
#include <map>
#include <numeric>

namespace emt {

namespace {

constexpr int kWave = 64, kQuad = 4, kMaxLg = 4;

// Rough cycles of one batch: its quads, its reduction and a fixed start.
int batch_cost(int quads, int lg) { return 60 + 40 * quads + 25 * lg; }

struct Batch {
  int lg, quads, cost;
  int first, count;  // rows, in the order below
};

// Batches of rows, longest first within a lane count, when a lane takes at
// most `most` entries (long rows take more once 2^kMaxLg lanes share them).
// `order` holds the rows by lane count, then length, the longest first; lg_of
// their lane counts.
void make_batches(const std::vector<RowSum> &rows, const std::vector<int> &order, const std::vector<int> &lg_of,
                  std::vector<Batch> &out) {
  out.clear();
  for (size_t k = 0; k < order.size(); ++k) {
    const int i = order[k], lg = lg_of[i];
    if (!out.empty() && out.back().lg == lg && out.back().count < (kWave >> lg)) {
      out.back().count++;
      continue;
    }
    const int per_lane = ((int)rows[i].e.size() + (1 << lg) - 1) >> lg;
    const int quads = std::max(1, (per_lane + kQuad - 1) / kQuad);
    out.push_back({lg, quads, batch_cost(quads, lg), (int)k, 1});
  }
}

// Batches to waves, dearest first onto the least loaded wave; returns the
// largest load.
int assign(const std::vector<Batch> &b, int waves, std::vector<int> &wave_of) {
  std::vector<int> idx(b.size()), load(waves, 0);
  std::iota(idx.begin(), idx.end(), 0);
  std::stable_sort(idx.begin(), idx.end(), [&](int x, int y) { return b[x].cost > b[y].cost; });
  wave_of.assign(b.size(), 0);
  for (int i : idx) {
    int w = 0;
    for (int k = 1; k < waves; ++k)
      if (load[k] < load[w]) w = k;
    wave_of[i] = w;
    load[w] += b[i].cost;
  }
  return *std::max_element(load.begin(), load.end());
}

}  // namespace

RowProgram schedule_rows(const std::vector<RowSum> &rows, int lanes, int pad_code, int pad_src,
                         const std::vector<int> *lg) {
  const int waves = lanes / kWave;
  std::vector<Batch> best, b;
  std::vector<int> best_wave, best_lg, w, lg_of(rows.size());
  int64_t best_cost = INT64_MAX;
  // a row's lanes grow with its length, so one order serves every choice of
  // `most`; given lane counts come first
  std::vector<int> order(rows.size());
  std::iota(order.begin(), order.end(), 0);
  auto lanes_of = [&](int most) {
    for (size_t i = 0; i < rows.size(); ++i) {
      const int cnt = (int)rows[i].e.size();
      int l = lg ? (*lg)[i] : 0;
      while (l < kMaxLg && (cnt + (1 << l) - 1) >> l > most) ++l;
      lg_of[i] = l;
    }
  };
  if (lg) lanes_of(16 * kQuad);
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
    if (lg && lg_of[x] != lg_of[y]) return lg_of[x] > lg_of[y];
    return rows[x].e.size() > rows[y].e.size();
  });
  if (!rows.empty())
    for (int q : {1, 2, 3, 4, 6, 8, 16}) {
      if (lg && q != 16) continue;
      if (!lg) lanes_of(q * kQuad);
      make_batches(rows, order, lg_of, b);
      // the slowest wave, and (LDS traffic) all quads
      int64_t quads = 0;
      for (const Batch &x : b) quads += x.quads;
      const int64_t cost = assign(b, waves, w) + 8 * quads;
      if (cost < best_cost) {
        best_cost = cost;
        best.swap(b);
        best_wave.swap(w);
        best_lg = lg_of;
      }
    }
  for (const RowSum &r : rows)
    if ((int)r.e.size() > kMaxRowEntries)
      throw Error{EMT_EINVAL, "a row of a component's sums has more than " + std::to_string(kMaxRowEntries) + " entries"};
  RowProgram p;
  p.lg = std::move(best_lg);
  p.meta.assign(waves + 1, 0);
  std::vector<int32_t> words;
  for (int w = 0; w < waves; ++w) {
    p.meta[w] = p.batches;
    for (size_t i = 0; i < best.size(); ++i) {
      if (best_wave[i] != w) continue;
      const Batch &b = best[i];
      words.push_back((int32_t)((uint32_t)p.quads | ((uint32_t)b.quads << 16) | ((uint32_t)b.lg << 24)));
      const size_t c0 = p.code.size();
      p.code.resize(c0 + (size_t)b.quads * kWave * kQuad, (uint16_t)pad_code);
      p.src.resize(c0 + (size_t)b.quads * kWave * kQuad, pad_src);
      p.row.resize(p.row.size() + kWave, 0xFFFF);
      const size_t r0 = p.row.size() - kWave;
      const int g = 1 << b.lg;
      for (int k = 0; k < b.count; ++k) {
        const RowSum &r = rows[order[b.first + k]];
        for (size_t e = 0; e < r.e.size(); ++e) {
          const int lane = k * g + (int)(e % g), slot = (int)(e / g);
          const int quad = slot / kQuad, s = slot % kQuad;
          p.code[c0 + ((size_t)quad * kWave + lane) * kQuad + s] = (uint16_t)r.e[e].first;
          p.src[c0 + (size_t)quad * kWave * kQuad + (size_t)(s / 2) * kWave * 2 + lane * 2 + (s & 1)] = r.e[e].second;
        }
        p.row[r0 + k * g + g - 1] = (uint16_t)r.row;
      }
      p.quads += b.quads;
      p.batches++;
    }
  }
  p.meta[waves] = p.batches;
  p.meta.insert(p.meta.end(), words.begin(), words.end());
  return p;
}

std::vector<ClosedSize> closed_sizes(const Symbolic &S, int dmax) {
  const int n = S.n;
  dmax = std::min(dmax, n);
  // A cluster of the leading ns nodes is a subtree of the elimination tree:
  // its root's parent (the first row below the root's pivot in L) lies in
  // the tail, and the tail nodes it touches are the root's column of L.
  std::vector<int64_t> size(n, 1);
  std::vector<int> parent(n, n);
  for (int i = 0; i < n; ++i) {
    if (S.lcol_ptr[i] < S.lcol_ptr[i + 1]) parent[i] = S.lcol_row[S.lcol_ptr[i]];
    if (parent[i] < n) size[parent[i]] += size[i];
  }
  std::vector<ClosedSize> out(dmax + 1);
  for (int d = 0; d <= dmax; ++d)
    for (int i = 0; i < n - d; ++i)
      if (parent[i] >= n - d) {
        out[d].q += size[i] * size[i];
        out[d].nn += size[i] * (S.lcol_ptr[i + 1] - S.lcol_ptr[i]);
      }
  return out;
}

ClosedPlan plan_closed(const Symbolic &S, const std::vector<int> &gpos, int d, int lanes) {
  const int n = S.n, ns = n - d;
  ClosedPlan P;
  P.d = d;
  P.ns = ns;
  std::vector<int> row_of(S.nnz());
  for (int i = 0; i < n; ++i)
    for (int q = S.lrow_ptr[i]; q < S.lrow_ptr[i + 1]; ++q) row_of[q] = i;
  // G's off-diagonal entries, each once, by position
  std::vector<int> pos = gpos;
  std::sort(pos.begin(), pos.end());
  pos.erase(std::unique(pos.begin(), pos.end()), pos.end());
  // clusters, by union over the entries of G_SS
  std::vector<int> root(ns);
  std::iota(root.begin(), root.end(), 0);
  auto find = [&](int i) {
    while (root[i] != i) i = root[i] = root[root[i]];
    return i;
  };
  for (int p : pos) {
    const int r = row_of[p], c = S.lrow_col[p];
    if (r < ns) root[find(c)] = find(r);
  }
  std::vector<std::vector<int>> mem;
  std::vector<int> cl_of(ns, -1), in_cl(ns, 0);
  for (int i = 0; i < ns; ++i) {
    const int f = find(i);
    if (cl_of[f] < 0) {
      cl_of[f] = (int)mem.size();
      mem.emplace_back();
    }
    mem[cl_of[f]].push_back(i);
  }
  std::stable_sort(mem.begin(), mem.end(),
                   [](const std::vector<int> &a, const std::vector<int> &b) { return a.size() > b.size(); });
  std::vector<int> qoff(mem.size());
  for (size_t c = 0; c < mem.size(); ++c) {
    qoff[c] = P.n_q;
    P.cluster.push_back((int32_t)mem[c].size());
    P.cluster.push_back(P.n_q);
    P.n_q += (int)(mem[c].size() * mem[c].size());
    for (size_t k = 0; k < mem[c].size(); ++k) {
      cl_of[mem[c][k]] = (int)c;
      in_cl[mem[c][k]] = (int)k;
    }
  }
  auto csize = [&](int c) { return (int)mem[c].size(); };
  for (int i = 0; i < ns; ++i) P.q_diag.push_back(qoff[cl_of[i]] + in_cl[i] * (csize(cl_of[i]) + 1));
  std::map<std::pair<int, int>, std::vector<std::pair<int, int>>> touch;  // (a, cluster) -> (L position, node)
  for (int p : pos) {
    const int r = row_of[p], c = S.lrow_col[p];
    if (r < ns) {
      const int cl = cl_of[r], s = csize(cl);
      P.q_off.push_back(p);
      P.q_off.push_back(qoff[cl] + in_cl[r] * s + in_cl[c]);
      P.q_off.push_back(p);
      P.q_off.push_back(qoff[cl] + in_cl[c] * s + in_cl[r]);
    } else if (c < ns) {
      touch[{r - ns, cl_of[c]}].push_back({p, c});
    } else {
      P.s_off.push_back(p);
      P.s_off.push_back((r - ns) * d + (c - ns));
      P.s_off.push_back(p);
      P.s_off.push_back((c - ns) * d + (r - ns));
    }
  }
  std::vector<std::vector<std::pair<int, int>>> groups_of(mem.size());  // cluster -> (a, first entry of N)
  P.n_ptr.push_back(0);
  std::vector<RowSum> fwd(d), bwd(ns);
  for (int a = 0; a < d; ++a) {
    fwd[a].row = a;
    fwd[a].e.push_back({ns + a, 1});
  }
  for (int i = 0; i < ns; ++i) {
    bwd[i].row = i;
    const int c = cl_of[i], s = csize(c);
    for (int k = 0; k < s; ++k) bwd[i].e.push_back({mem[c][k], -(qoff[c] + in_cl[i] * s + k) - 1});
  }
  int grp = 0;
  for (auto &t : touch) {
    const int a = t.first.first, c = t.first.second, s = csize(c);
    groups_of[c].push_back({a, P.n_n});
    for (auto &e : t.second) {
      P.n_adj.push_back(e.first);
      P.n_adj.push_back(qoff[c] + in_cl[e.second] * s);
    }
    for (int k = 0; k < s; ++k) {
      fwd[a].e.push_back({mem[c][k], P.value_n(P.n_n)});
      bwd[mem[c][k]].e.push_back({n + 1 + ns + a, P.value_n(P.n_n)});
      P.n_grp.push_back(grp);
      P.n_col.push_back(k);
      P.n_n++;
    }
    P.n_ptr.push_back((int32_t)P.n_adj.size() / 2);
    ++grp;
  }
  for (RowSum &r : bwd)
    for (auto &e : r.e)
      if (e.second < 0) e.second = P.value_q(-e.second - 1);
  // S_ab = G_ab + sum over the clusters both touch of N_ak G_kb
  std::map<int, std::vector<std::pair<int, int>>> terms;
  for (auto &t : touch) {
    const int b = t.first.first, c = t.first.second;
    for (auto &ga : groups_of[c])
      for (auto &e : t.second) terms[ga.first * d + b].push_back({ga.second + in_cl[e.second], e.first});
  }
  P.s_ptr.push_back(0);
  for (auto &t : terms) {
    P.s_key.push_back(t.first);
    for (auto &e : t.second) {
      P.s_term.push_back(e.first);
      P.s_term.push_back(e.second);
    }
    P.s_ptr.push_back((int32_t)P.s_term.size() / 2);
  }
  P.fwd = schedule_rows(fwd, lanes, n, 0);
  P.bwd = schedule_rows(bwd, lanes, n, 0);
  return P;
}

}  // namespace emt
