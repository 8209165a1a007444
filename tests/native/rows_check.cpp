// Host-side replay of the row-by-row factorisation schedule and of the split
// block storage (built by tests/test_host_rows.py with sanitizers).  The
// chunks are run as the kernel runs them: rows of a chunk dealt to the lane
// groups, each row's steps applied in its group's buffer, finished rows written
// to storage.  Checked: every row once, level by level; buffers of concurrent
// groups disjoint and inside the area; every block, target and pivot row in
// range and read only after the pass that writes it; the L+U values outside the
// tail, and the tail rows' partial sums, equal a plain block LU of the pattern
// to 1e-9 (random diagonally dominant values); the solve schedules' first
// positions, pivot inverses and transposed positions follow the storage.
// The wavefront tasks of the same rows are replayed after it: tasks in level
// order, each step's pivot of a lower level that its record names, every row
// once, buffers and records within a wavefront's share, and the
// same factors.
// Usage: rows_check NET TAIL_MAX SLICE THREADS BUFFER_BLOCKS BUDGET
#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <fstream>
#include <random>
#include <string>
#include <vector>

#include "sable_pf.h"
#include "symbolic.h"

using namespace sable;
using B = std::array<double, 4>;
static int g_fail = 0;
#define CHECK(c, ...) do { if (!(c)) { if (g_fail++ < 10) { std::printf(__VA_ARGS__); std::printf("\n"); } } } while (0)

static B mul(const B& x, const B& y) {
  return {x[0] * y[0] + x[1] * y[2], x[0] * y[1] + x[1] * y[3], x[2] * y[0] + x[3] * y[2], x[2] * y[1] + x[3] * y[3]};
}
static B inv(const B& x) {
  const double d = x[0] * x[3] - x[1] * x[2];
  return {x[3] / d, -x[1] / d, -x[2] / d, x[0] / d};
}
static B sub(const B& x, const B& y) { return {x[0] - y[0], x[1] - y[1], x[2] - y[2], x[3] - y[3]}; }

int main(int argc, char** argv) {
  if (argc != 7) return 2;
  std::ifstream in(argv[1]);
  int n, m;
  in >> n >> m;
  std::vector<int32_t> bt(n), f(m), t(m), yrp, yci;
  std::vector<double> r(m), x(m), bc(m), g, b;
  for (auto& v : bt) in >> v;
  for (int k = 0; k < m; ++k) in >> f[k] >> t[k] >> r[k] >> x[k] >> bc[k];
  const int tail_max = std::atoi(argv[2]), slice = std::atoi(argv[3]), threads = std::atoi(argv[4]);
  const int64_t area = std::atoll(argv[5]);
  const int budget = std::atoi(argv[6]);
  std::string err;
  if (ybus_from_branches(n, m, f.data(), t.data(), r.data(), x.data(), bc.data(), yrp, yci, g, b, err) < 0) return 2;
  Symbolic S;
  if (analyze(n, bt.data(), yrp.data(), yci.data(), g.data(), b.data(), S, err, tail_max) != 0) return 2;
  const LuStorage st = storage_split(S);
  const int nb = S.nb, nz = S.nnzb(), tb = S.tail_base;
  std::vector<int> seen(nz, 0);
  for (int p = 0; p < nz; ++p) {
    CHECK(st.pos[p] >= 0 && st.pos[p] < nz, "storage of %d", p);
    seen[st.pos[p]]++;
  }
  for (int v : seen) CHECK(v == 1, "storage index used %d times", v);

  RowChunks R;
  if (build_row_chunks(S, st, slice, threads, area, budget, R, err) != 0) {
    std::printf("refused: %s\n", err.c_str());
    return 3;
  }
  CHECK(R.max_ints <= budget && R.max_buffer <= area, "chunk of %d words, buffers of %lld blocks", R.max_ints, (long long)R.max_buffer);

  // values and the plain elimination, row by row in pivot order
  std::mt19937 rng(7);
  std::uniform_real_distribution<double> U(-1, 1);
  std::vector<B> A(nz), ref, lu(nz);
  for (int a = 0; a < nb; ++a)
    for (int p = S.rp[a]; p < S.rp[a + 1]; ++p)
      for (int c = 0; c < 4; ++c) A[p][c] = U(rng) + ((S.ci[p] == a && (c == 0 || c == 3)) ? 4.0 + S.rp[a + 1] - S.rp[a] : 0.0);
  ref = A;
  for (int a = 0; a < nb; ++a) {
    std::vector<int> at(nb, -1);
    for (int p = S.rp[a]; p < S.rp[a + 1]; ++p) at[S.ci[p]] = p;
    for (int p = S.rp[a]; p < S.diag[a]; ++p) {
      const int k = S.ci[p];
      if (k >= tb) break;
      for (int q = S.diag[k] + 1; q < S.rp[k + 1]; ++q) ref[at[S.ci[q]]] = sub(ref[at[S.ci[q]]], mul(ref[p], ref[q]));
    }
    if (a >= tb) continue;   // rows outside the tail: U scaled by the inverted pivot block
    for (int p = S.diag[a] + 1; p < S.rp[a + 1]; ++p) ref[p] = mul(inv(ref[S.diag[a]]), ref[p]);
  }

  std::vector<int> done(nb, -1);
  const int nch = (int)R.ptr.size() - 1;
  for (int c = 0; c < nch; ++c) {
    const int32_t* h = &R.blob[R.ptr[c]];
    const int nrow = h[0], nstep = h[1], lg = h[2] & 255, lsw = h[2] >> 8;
    const int32_t* rw = h + 4;
    const int32_t* sp = rw + 8 * (nrow + 1);
    const int32_t* tg = sp + 4 * (nstep + 1);
    CHECK(R.ptr[c] % 4 == 0 && R.ptr[c + 1] % 4 == 0, "chunk %d alignment", c);
    const int lanes = 1 << lg, ng = threads >> lg;
    CHECK(lanes >= slice && lanes <= threads && ng >= 1, "chunk %d: %d lanes per row", c, lanes);
    CHECK(lanes <= 64 ? (1 << lsw) == slice : (lanes / 64) * (1 << lsw) == slice, "chunk %d: scenarios per wavefront", c);
    std::vector<B> buf(area);
    std::vector<std::pair<int64_t, int64_t>> use(ng, {0, 0});   // [first, end) of every group's buffer
    for (int i = 0; i < nrow; ++i) {
      const int32_t *r0 = rw + 8 * i, *r1 = r0 + 4;
      const int a = r1[0], nl = r1[3] & (kRowPv - 1), s0 = r0[3], s1 = r0[8 + 3];
      CHECK(a >= 0 && a < nb && done[a] < 0, "row %d twice", a);
      if (a < 0 || a >= nb) continue;
      CHECK(r0[0] == S.blk_bus[a] && r0[1] == S.rp[a + 1] - S.rp[a] && nl == S.diag[a] - S.rp[a], "row %d record", a);
      CHECK(((r1[3] & kRowFinal) != 0) == (a < tb) && ((r1[3] & kRowPv) != 0) == (bt[S.blk_bus[a]] == PF_BUS_PV), "row %d flags", a);
      for (int j = 0; j < r0[1]; ++j)
        CHECK((j <= nl ? r1[1] + j : r1[2] + j - nl - 1) == st.pos[S.rp[a] + j], "row %d block %d storage", a, j);
      CHECK(st.dinv[a] == r1[1] + nl, "row %d pivot storage", a);
      int nsteps = 0;
      for (int p = S.rp[a]; p < S.diag[a]; ++p) nsteps += S.ci[p] < tb;
      CHECK(s1 - s0 == nsteps, "row %d: %d steps of %d", a, s1 - s0, nsteps);
      std::vector<B> W(r0[1]);
      for (int j = 0; j < r0[1]; ++j) W[j] = A[S.rp[a] + j];
      {
        CHECK(r0[2] >= 0 && r0[2] + r0[1] <= area, "row %d buffer", a);
        auto& u = use[i % ng];
        if (u.second == u.first) u = {r0[2], r0[2] + r0[1]};
        CHECK(r0[2] == u.first && r0[2] + r0[1] <= u.second, "row %d: its group's buffer", a);
      }
      for (int k = s0; k < s1; ++k) {
        const int32_t* q = sp + 4 * k;
        const int nt = q[4 + 3] - q[3], piv = q[1];
        CHECK(q[0] == k - s0 && piv == S.ci[S.rp[a] + q[0]], "row %d step %d", a, k - s0);
        CHECK(done[piv] >= 0 && done[piv] < c, "row %d reads row %d in pass %d, written in %d", a, piv, c, done[piv]);
        CHECK(nt >= 1 && q[2] == st.pos[S.diag[piv] + 1] && nt == S.rp[piv + 1] - S.diag[piv] - 1, "row %d step %d pivot row", a, k - s0);
        for (int j = 0; j < nt; ++j) {
          const int w = tg[q[3] + j];
          CHECK(w > q[0] && w < r0[1] && S.ci[S.rp[a] + w] == S.ci[S.diag[piv] + 1 + j], "row %d step %d target %d", a, k - s0, j);
          W[w] = sub(W[w], mul(W[q[0]], lu[q[2] + j]));
        }
      }
      if (a < tb) {
        W[nl] = inv(W[nl]);
        for (int j = nl + 1; j < r0[1]; ++j) W[j] = mul(W[nl], W[j]);
      }
      for (int j = 0; j < r0[1]; ++j) lu[st.pos[S.rp[a] + j]] = W[j];
      done[a] = c;
    }
    std::sort(use.begin(), use.end());
    for (size_t i = 1; i < use.size(); ++i)
      CHECK(use[i].first >= use[i - 1].second || use[i].first == use[i].second, "chunk %d: buffers overlap", c);
  }
  double worst = 0;
  for (int a = 0; a < nb; ++a) {
    CHECK(done[a] >= 0, "row %d missing", a);
    for (int p = S.rp[a]; p < S.rp[a + 1]; ++p) {
      const B want = S.ci[p] == a && a < tb ? inv(ref[p]) : ref[p];
      for (int c = 0; c < 4; ++c) worst = std::max(worst, std::fabs(lu[st.pos[p]][c] - want[c]));
    }
  }
  CHECK(worst < 1e-9, "factors differ by %g", worst);

  // ---- wavefront tasks, with a sixteenth of the areas each
  const int waves = threads / 64;
  const int64_t share = area * slice / waves;
  const int meta = std::min(kFlowMaxWords, budget / waves / 4 * 4);
  FlowTasks F;
  if (build_flow_tasks(S, st, waves, share, meta, F, err) != 0) {
    std::printf("flow refused: %s\n", err.c_str());
  } else {
    std::vector<B> fl(nz);
    std::vector<int> lev(nb, -1), cover(nb, 0), count(F.per_level.size(), 0);
    int last = 0;
    CHECK(F.max_ints <= meta, "task record of %d words", F.max_ints);
    for (int k = 0; k < F.n_tasks(); ++k) {
      const int32_t* c = &F.blob[F.task[2 * k]];
      const int words = F.task[2 * k + 1];
      const int nrow = c[0], lanes = 1 << c[1], h = c[2], most = c[3];
      CHECK(F.task[2 * k] % 4 == 0 && F.task[2 * k] + 4 * words <= (int)F.blob.size(), "task %d record", k);
      CHECK(h >= last && h < (int)F.per_level.size(), "task %d of level %d after %d", k, h, last);
      CHECK(lanes <= 64 && nrow >= 1 && nrow * lanes <= 64, "task %d geometry", k);
      last = h;
      count[h]++;
      const int32_t* sp = c + 4 + 8 * nrow;
      const int32_t* lr = c + 4 + 8 * (nrow - 1);
      const int nsteps = lr[3] + (lr[1] >> 16);
      const unsigned char* tg = reinterpret_cast<const unsigned char*>(sp + 4 * nsteps);
      int blocks = 0, longest = 0;
      for (int i = 0; i < nrow; ++i) {
        const int32_t *r0 = c + 4 + 8 * i, *r1 = r0 + 4;
        const int a = r1[0], n = r0[1] & 0xffff, ns = r0[1] >> 16, nl = r1[3] & (kRowPv - 1);
        int outer = 0;
        for (int p = S.rp[a]; p < S.diag[a]; ++p) outer += S.ci[p] < tb;
        CHECK(a >= 0 && a < nb && r0[0] == S.blk_bus[a] && n == S.rp[a + 1] - S.rp[a] && ns == outer && nl == S.diag[a] - S.rp[a], "task row %d", a);
        CHECK(((r1[3] & kRowFinal) != 0) == (a < tb), "task row %d: final", a);
        CHECK(((r1[3] & kRowPv) != 0) == (bt[S.blk_bus[a]] == PF_BUS_PV), "task row %d flags", a);
        CHECK(r0[2] == blocks, "task row %d buffer", a);
        blocks += n;
        longest = std::max(longest, ns);
        cover[a]++;
        lev[a] = h;
        for (int j = 0; j < n; ++j) CHECK((j <= nl ? r1[1] + j : r1[2] + j - nl - 1) == st.pos[S.rp[a] + j], "task row %d block %d", a, j);
        std::vector<B> W(n);
        for (int j = 0; j < n; ++j) W[j] = A[S.rp[a] + j];
        for (int q = 0; q < ns; ++q) {
          const int32_t* x = sp + 4 * (r0[3] + q);
          const int piv = x[1], nu = (x[0] >> 8) & 255, blk = x[0] & 255;
          CHECK(blk == q && piv == S.ci[S.rp[a] + q] && nu == S.rp[piv + 1] - S.diag[piv] - 1 && nu >= 1, "task row %d step %d", a, q);
          CHECK(lev[piv] >= 0 && lev[piv] < h && (x[0] >> 16) == lev[piv], "task row %d: level of pivot %d", a, piv);
          CHECK(x[2] == st.pos[S.diag[piv] + 1], "task row %d: pivot row", a);
          for (int j = 0; j < nu; ++j) {
            const int w = tg[x[3] + j];
            CHECK(x[3] + j < 4 * (4 * words - (int)(sp + 4 * nsteps - c)) && w > blk && w < n, "task row %d target", a);
            CHECK(S.ci[S.rp[a] + w] == S.ci[S.diag[piv] + 1 + j], "task row %d step %d target %d", a, q, j);
            W[w] = sub(W[w], mul(W[blk], fl[x[2] + j]));
          }
        }
        if (a < tb) {
          W[nl] = inv(W[nl]);
          for (int j = nl + 1; j < n; ++j) W[j] = mul(W[nl], W[j]);
        }
        for (int j = 0; j < n; ++j) fl[st.pos[S.rp[a] + j]] = W[j];
      }
      CHECK(blocks <= share && longest == most, "task %d: buffer of %d blocks, %d steps", k, blocks, most);
    }
    for (size_t h = 0; h < count.size(); ++h) CHECK(count[h] == F.per_level[h], "level %zu: %d tasks", h, count[h]);
    for (int a = 0; a < nb; ++a) {
      CHECK(cover[a] == 1, "row %d in %d tasks", a, cover[a]);
      for (int p = S.rp[a]; p < S.rp[a + 1]; ++p)
        for (int c = 0; c < 4; ++c) CHECK(fl[st.pos[p]][c] == lu[st.pos[p]][c], "row %d: task values", a);
    }
    std::printf("flow tasks %d words %d ", F.n_tasks(), F.max_ints);
  }

  LevelChunks C;
  if (build_level_chunks(S, budget, C, err, &st) != 0) return 3;
  auto solves = [&](const std::vector<int32_t>& ptr, const std::vector<int32_t>& blob, bool lower, bool pairs) {
    for (size_t c = 0; c + 1 < ptr.size(); ++c) {
      const int32_t* h = &blob[ptr[c]];
      const int32_t* cols = h + 4 + 4 * (h[0] + 1);
      for (int i = 0; i < h[0]; ++i) {
        const int32_t* q = h + 4 + 4 * i;
        const int a = q[0], p0 = lower ? S.rp[a] : S.diag[a] + 1, p1 = lower ? S.diag[a] : S.rp[a + 1];
        CHECK(q[4 + 3] - q[3] == p1 - p0 && q[2] == st.dinv[a], "solve row %d", a);
        for (int p = p0; p < p1; ++p) {
          const int j = q[3] + p - p0;
          CHECK(st.pos[p] == q[1] + p - p0, "solve row %d: position", a);
          CHECK(cols[pairs ? 2 * j : j] == S.ci[p] && (!pairs || cols[2 * j + 1] == st.pos[S.mirror[p]]), "solve row %d: column", a);
        }
      }
    }
  };
  solves(C.fs_ptr, C.fs_blob, true, false);
  solves(C.bs_ptr, C.bs_blob, false, false);
  solves(C.ut_ptr, C.ut_blob, true, true);
  solves(C.lt_ptr, C.lt_blob, false, true);
  for (int l = 0, q = 0; l < S.tail_t; ++l)
    for (int p = S.rp[tb + l]; p < S.tail_split[l]; ++p, ++q)
      CHECK(C.tt_pairs[2 * q] == S.ci[p] && C.tt_pairs[2 * q + 1] == st.pos[S.mirror[p]], "tail row %d: transposed term", l);
  CHECK(C.f_ptr.empty(), "factor tasks with split storage");
  std::printf("rows %d chunks %d words %d buffer %lld worst %.1e violations %d\n", nb, nch, R.max_ints,
              (long long)R.max_buffer, worst, g_fail);
  return g_fail ? 1 : 0;
}
