// Host check of the closed-form plan (csrc/closed.cpp), built with the
// address and undefined-behaviour sanitizers by tests/test_closed_host.py:
// random networks, every cut from none to the whole component and the three
// workgroup sizes; the plan's numbers are formed from its lists, its row
// programs run lane by lane as the kernels run them, and the result is
// compared with a dense solve.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "closed.h"

using namespace emt;

static void require(bool ok, const char *what) {
  if (ok) return;
  std::printf("FAILED: %s\n", what);
  std::exit(1);
}

using Mat = std::vector<std::vector<double>>;

static Mat inverse(Mat a) {
  const int n = (int)a.size();
  for (int p = 0; p < n; ++p) {
    const double d = 1.0 / a[p][p];
    for (int i = 0; i < n; ++i)
      for (int j = 0; j < n; ++j)
        if (i != p && j != p) a[i][j] -= a[i][p] * a[p][j] * d;
    for (int i = 0; i < n; ++i)
      if (i != p) {
        a[i][p] *= -d;
        a[p][i] *= d;
      }
    a[p][p] = d;
  }
  return a;
}

// Sum of every row of a program: lanes add up their quads, a row's lanes in
// a group end at its last lane.
template <class Term>
static void run(const RowProgram &p, int lanes, Term term, std::vector<double> &out, std::vector<int> &wrote) {
  const int waves = lanes / 64;
  require((int)p.meta.size() == waves + 1 + p.batches && p.meta[0] == 0 && p.meta[waves] == p.batches, "batch table");
  require((int)p.code.size() == p.quads * 256 && (int)p.row.size() == p.batches * 64 &&
              (int)p.src.size() == p.quads * 256, "program sizes");
  for (int w = 0; w < waves; ++w)
    for (int b = p.meta[w]; b < p.meta[w + 1]; ++b) {
      const uint32_t m = (uint32_t)p.meta[waves + 1 + b];
      const int q0 = m & 0xFFFF, nq = (m >> 16) & 0xFF, lg = m >> 24;
      require(lg <= 4 && nq >= 1 && q0 + nq <= p.quads, "batch word");
      for (int lane = 0; lane < 64; ++lane) {
        const int row = p.row[b * 64 + lane];
        if (row == 0xFFFF) continue;
        require((lane & ((1 << lg) - 1)) == (1 << lg) - 1, "a row ends in its group's last lane");
        double s = 0.0;
        for (int l = lane - (1 << lg) + 1; l <= lane; ++l)
          for (int q = q0; q < q0 + nq; ++q)
            for (int k = 0; k < 4; ++k)
              s += term(p.code[(q * 64 + l) * 4 + k], p.src[q * 256 + (k / 2) * 128 + l * 2 + (k & 1)]);
        require(row < (int)out.size(), "row in range");
        out[row] = s;
        wrote[row]++;
      }
    }
}

int main() {
  int checks = 0;
  double worst = 0.0;
  for (int n : {1, 2, 9, 37, 90})
    for (int trial = 0; trial < 2; ++trial) {
      // a random tree plus extra branches, some to ground
      std::srand(n * 10 + trial);
      std::vector<int> k, m, kind;
      std::vector<double> R, L, C;
      auto add = [&](int a, int b) {
        k.push_back(a);
        m.push_back(b);
        kind.push_back(EMT_R);
        R.push_back(0.5 + (std::rand() % 1000) / 100.0);
        L.push_back(1.0);
        C.push_back(1.0);
      };
      for (int i = 0; i < n; ++i) {
        add(i, -1);
        if (i > 0) add(i, std::rand() % i);
      }
      for (int e = 0; e < n / 2; ++e) {
        const int a = std::rand() % n, b = std::rand() % n;
        if (a != b) add(a, b);
      }
      emt_net net{};
      net.n_nodes = n;
      net.n_branches = (int)k.size();
      net.k = k.data();
      net.m = m.data();
      net.kind = kind.data();
      net.R = R.data();
      net.L = L.data();
      net.C = C.data();
      net.n_rec = n;
      emt_sim sim{};
      sim.dt = 1e-5;
      sim.n_steps = 1;
      sim.dense_tail = -1;
      const Analysis A = analyze(&net, 1, sim);
      require(A.items.size() == 1, "one component");
      const Item &it = A.items[0];
      const Symbolic &S = A.syms[it.sym];
      std::vector<int> gpos;
      for (int p : it.gpos)
        if (p >= 0) gpos.push_back(p);
      // G by L position and dense
      std::vector<double> low(S.nnz(), 0.0), diag(n, 0.0);
      Mat G(n, std::vector<double>(n, 0.0));
      for (int j = 0; j < it.n_br; ++j) {
        const double g = 1.0 / R[it.br[j]];
        const int a = it.bk[j], b = it.bm[j];
        for (int e : {a, b})
          if (e >= 0) {
            diag[e] += g;
            G[e][e] += g;
          }
        if (a >= 0 && b >= 0) {
          low[it.gpos[j]] -= g;
          G[a][b] -= g;
          G[b][a] -= g;
        }
      }
      const Mat X = inverse(G);
      std::vector<double> r(n), ref(n, 0.0);
      for (int i = 0; i < n; ++i) r[i] = (std::rand() % 2001 - 1000) / 500.0;
      for (int i = 0; i < n; ++i)
        for (int j = 0; j < n; ++j) ref[i] += X[i][j] * r[j];
      const std::vector<ClosedSize> sizes = closed_sizes(S, n);
      require((int)sizes.size() == n + 1, "one size per cut");
      for (int lanes : {64, 256, 512})
        for (int d = 0; d <= n; d += 1 + (d > 4 ? 6 : 0)) {
          const ClosedPlan P = plan_closed(S, gpos, d, lanes);
          const int ns = n - d;
          require(P.d == d && P.ns == ns && P.n_q == sizes[d].q && P.n_n == sizes[d].nn, "sizes");
          std::vector<double> V(2 + P.n_n + P.n_q, 0.0);
          V[1] = 1.0;
          for (int i = 0; i < ns; ++i) V[P.value_q(P.q_diag[i])] = diag[i];
          for (size_t e = 0; e < P.q_off.size(); e += 2) V[P.value_q(P.q_off[e + 1])] = low[P.q_off[e]];
          for (size_t c = 0; c < P.cluster.size(); c += 2) {
            const int s = P.cluster[c], o = P.cluster[c + 1];
            require(c == 0 || s <= P.cluster[c - 2], "largest clusters first");
            Mat a(s, std::vector<double>(s));
            for (int i = 0; i < s; ++i)
              for (int j = 0; j < s; ++j) a[i][j] = V[P.value_q(o + i * s + j)];
            a = inverse(a);
            for (int i = 0; i < s; ++i)
              for (int j = 0; j < s; ++j) V[P.value_q(o + i * s + j)] = a[i][j];
          }
          for (int e = 0; e < P.n_n; ++e) {
            double s = 0.0;
            for (int q = P.n_ptr[P.n_grp[e]]; q < P.n_ptr[P.n_grp[e] + 1]; ++q)
              s += low[P.n_adj[2 * q]] * V[P.value_q(P.n_adj[2 * q + 1] + P.n_col[e])];
            V[P.value_n(e)] = -s;
          }
          Mat W(d, std::vector<double>(d, 0.0));
          for (int a = 0; a < d; ++a) W[a][a] = diag[ns + a];
          for (size_t e = 0; e < P.s_off.size(); e += 2) W[P.s_off[e + 1] / d][P.s_off[e + 1] % d] = low[P.s_off[e]];
          for (size_t q = 0; q < P.s_key.size(); ++q)
            for (int e = P.s_ptr[q]; e < P.s_ptr[q + 1]; ++e)
              W[P.s_key[q] / d][P.s_key[q] % d] += V[P.value_n(P.s_term[2 * e])] * low[P.s_term[2 * e + 1]];
          W = inverse(W);
          // right-hand side, its zero, the solution, its zero
          std::vector<double> xr(2 * (n + 1), 0.0), c(d, 0.0), x(ns, 0.0);
          for (int i = 0; i < n; ++i) xr[i] = r[i];
          auto term = [&](int code, int src) {
            require(code < (int)xr.size() && src < (int)V.size(), "code and value in range");
            return V[src] * xr[code];
          };
          std::vector<int> wc(d, 0), wx(ns, 0);
          run(P.fwd, lanes, term, c, wc);
          for (int a = 0; a < d; ++a)
            for (int b = 0; b < d; ++b) xr[n + 1 + ns + a] += W[a][b] * c[b];
          run(P.bwd, lanes, term, x, wx);
          for (int v : wc) require(v == 1, "every tail row once");
          for (int v : wx) require(v == 1, "every leading row once");
          for (int i = 0; i < n; ++i) {
            const double got = i < ns ? x[i] : xr[n + 1 + i];
            worst = std::max(worst, std::fabs(got - ref[i]));
          }
          ++checks;
        }
    }
  std::printf("checks %d worst %.3g\n", checks, worst);
  // conductances in [0.1, 2], every node grounded: |x| stays below 100 and
  // the condition number below 1e4
  require(worst < 1e-9, "solution");
  std::printf("ok\n");
  return 0;
}
