// Host-side check of the launch plan of HBM-resident templates (built by
// tests/test_host_plan.py with sanitizers): the network is analysed and planned
// exactly as pf_template_build does, the parts of a workgroup's LDS are checked
// to lie one behind the other inside it, and the plan's factorisation schedule
// is replayed on random diagonally dominant values: every row once, pivots read
// only after the pass (level) that writes them, buffers and records inside their
// areas, and the factors equal a plain block LU of the pattern to 1e-9.
// Usage: plan_check NET fp64|mixed BATCH THREADS
// prints: path tasks|rows|levels slice S y Y lds BYTES ... violations N
#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <random>
#include <string>
#include <vector>

#include "hbm_plan.h"
#include "sable_pf.h"

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
static void sub(B& x, const B& y) { for (int c = 0; c < 4; ++c) x[c] -= y[c]; }

struct Replay {
  const Symbolic& S;
  const LuStorage& st;
  std::vector<B> A, lu;
  std::vector<int> done;   // pass that wrote a row, -1: none
  Replay(const Symbolic& S_, const LuStorage& st_) : S(S_), st(st_), A(S_.nnzb()), lu(S_.nnzb()), done(S_.nb, -1) {
    std::mt19937 rng(7);
    std::uniform_real_distribution<double> U(-1, 1);
    for (int a = 0; a < S.nb; ++a)
      for (int p = S.rp[a]; p < S.rp[a + 1]; ++p)
        for (int c = 0; c < 4; ++c)
          A[p][c] = U(rng) + ((S.ci[p] == a && (c == 0 || c == 3)) ? 4.0 + S.rp[a + 1] - S.rp[a] : 0.0);
  }
  int steps(int a) const {
    int n = 0;
    for (int p = S.rp[a]; p < S.diag[a]; ++p) n += S.ci[p] < S.tail_base;
    return n;
  }
  // one row by its records r (eight words), steps (block, pivot, storage of the
  // pivot's U part, number of them) and targets
  struct Step { int blk, piv, u, n; };
  void row(const int32_t* r, int pass, const std::vector<Step>& steps_, const std::vector<int>& tgt) {
    const int a = r[4], n = r[1] & 0xffff, nl = r[7] & (kRowPv - 1);
    CHECK(a >= 0 && a < S.nb && done[a] < 0, "row %d twice", a);
    if (a < 0 || a >= S.nb) return;
    CHECK(r[0] == S.blk_bus[a] && n == S.rp[a + 1] - S.rp[a] && nl == S.diag[a] - S.rp[a], "row %d record", a);
    CHECK(((r[7] & kRowFinal) != 0) == (a < S.tail_base), "row %d: final", a);
    CHECK(((r[7] & kRowPv) != 0) == (S.bus_type[S.blk_bus[a]] == PF_BUS_PV), "row %d: PV", a);
    CHECK((int)steps_.size() == steps(a), "row %d: %zu steps", a, steps_.size());
    std::vector<B> W(A.begin() + S.rp[a], A.begin() + S.rp[a + 1]);
    size_t t = 0;
    for (const Step& q : steps_) {
      CHECK(q.piv == S.ci[S.rp[a] + q.blk] && done[q.piv] >= 0 && done[q.piv] < pass, "row %d reads row %d", a, q.piv);
      CHECK(q.n == S.rp[q.piv + 1] - S.diag[q.piv] - 1 && q.u == st.pos[S.diag[q.piv] + 1], "row %d: pivot row %d", a, q.piv);
      for (int j = 0; j < q.n; ++j, ++t) {
        const int w = tgt[t];
        CHECK(w > q.blk && w < n && S.ci[S.rp[a] + w] == S.ci[S.diag[q.piv] + 1 + j], "row %d: target", a);
        sub(W[w], mul(W[q.blk], lu[q.u + j]));
      }
    }
    if (a < S.tail_base) {
      W[nl] = inv(W[nl]);
      for (int j = nl + 1; j < n; ++j) W[j] = mul(W[nl], W[j]);
    }
    for (int j = 0; j < n; ++j) {
      const int at = j <= nl ? r[5] + j : r[6] + j - nl - 1;
      CHECK(at == st.pos[S.rp[a] + j], "row %d block %d: storage", a, j);
      lu[at] = W[j];
    }
    done[a] = pass;
  }
  void finish() {
    std::vector<B> ref = A;
    std::vector<int> at(S.nb, -1);
    double worst = 0;
    for (int a = 0; a < S.nb; ++a) {
      CHECK(done[a] >= 0, "row %d missing", a);
      for (int p = S.rp[a]; p < S.rp[a + 1]; ++p) at[S.ci[p]] = p;
      for (int p = S.rp[a]; p < S.diag[a] && S.ci[p] < S.tail_base; ++p)
        for (int q = S.diag[S.ci[p]] + 1; q < S.rp[S.ci[p] + 1]; ++q) sub(ref[at[S.ci[q]]], mul(ref[p], ref[q]));
      if (a < S.tail_base) {
        ref[S.diag[a]] = inv(ref[S.diag[a]]);
        for (int p = S.diag[a] + 1; p < S.rp[a + 1]; ++p) ref[p] = mul(ref[S.diag[a]], ref[p]);
      }
      for (int p = S.rp[a]; p < S.rp[a + 1]; ++p)
        for (int c = 0; c < 4; ++c) worst = std::max(worst, std::fabs(lu[st.pos[p]][c] - ref[p][c]));
    }
    CHECK(worst < 1e-9, "factors differ by %g", worst);
  }
};

static void replay_tasks(Replay& R, const HbmPlan& P, int waves) {
  const FlowTasks& F = P.flow;
  std::vector<int> count(F.per_level.size(), 0);
  int last = 0;
  for (int k = 0; k < F.n_tasks(); ++k) {
    const int32_t* c = &F.blob[F.task[2 * k]];
    const int words = 4 * F.task[2 * k + 1], nrow = c[0], lanes = 1 << c[1], h = c[2];
    CHECK(F.task[2 * k] % 4 == 0 && F.task[2 * k] + words <= (int)F.blob.size(), "task %d: record", k);
    CHECK(words <= P.flow_meta, "task %d: %d words in an area of %d", k, words, P.flow_meta);
    CHECK(nrow >= 1 && lanes <= 64 && nrow * lanes <= 64, "task %d: geometry", k);
    CHECK(h >= last && h < (int)count.size(), "task %d: level", k);
    last = h;
    count[h]++;
    const int32_t* sp = c + 4 + 8 * nrow;
    const int32_t* lr = c + 4 + 8 * (nrow - 1);
    const int nsteps = lr[3] + (lr[1] >> 16);
    const unsigned char* tg = reinterpret_cast<const unsigned char*>(sp + 4 * nsteps);
    const int room = (int)(reinterpret_cast<const unsigned char*>(c + words) - tg);
    int blocks = 0, most = 0;
    for (int i = 0; i < nrow; ++i) {
      const int32_t* r = c + 4 + 8 * i;
      CHECK(r[2] == blocks, "task %d: buffer", k);
      blocks += r[1] & 0xffff;
      most = std::max(most, r[1] >> 16);
      std::vector<Replay::Step> steps;
      std::vector<int> tgt;
      for (int q = 0; q < r[1] >> 16; ++q) {
        const int32_t* x = sp + 4 * (r[3] + q);
        const int nu = (x[0] >> 8) & 255;
        steps.push_back({x[0] & 255, x[1], x[2], nu});
        CHECK(R.done[x[1]] == (x[0] >> 16) + 1, "task %d: level of pivot %d", k, x[1]);
        CHECK(x[3] + nu <= room, "task %d: targets", k);
        for (int j = 0; j < nu; ++j) tgt.push_back(tg[x[3] + j]);
      }
      R.row(r, h + 1, steps, tgt);
    }
    CHECK(blocks <= P.flow_buf && most == c[3], "task %d: %d blocks in a buffer of %d", k, blocks, P.flow_buf);
  }
  for (size_t h = 0; h < count.size(); ++h) CHECK(count[h] == F.per_level[h], "level %zu: %d tasks", h, count[h]);
  // records, the counts of the levels and the next task in the metadata area
  CHECK(waves * P.flow_meta + (int)count.size() + 1 <= P.chunk_ints, "records and counts beyond the metadata area");
}

static void replay_rows(Replay& R, const HbmPlan& P, int threads, size_t tsz) {
  const RowChunks& C = P.row_chunks;
  const int64_t area = (int64_t)(P.area / (4 * tsz * P.slice));
  for (size_t k = 0; k + 1 < C.ptr.size(); ++k) {
    const int32_t* h = &C.blob[C.ptr[k]];
    const int nrow = h[0], nstep = h[1], lg = h[2] & 255, lsw = h[2] >> 8, lanes = 1 << lg, ng = threads >> lg;
    const int32_t* rw = h + 4;
    const int32_t* sp = rw + 8 * (nrow + 1);
    const int32_t* tg = sp + 4 * (nstep + 1);
    CHECK(C.ptr[k] % 4 == 0 && C.ptr[k + 1] - C.ptr[k] <= P.chunk_ints, "chunk %zu beyond the metadata area", k);
    CHECK(lanes >= P.slice && ng >= 1, "chunk %zu: %d lanes per row", k, lanes);
    CHECK(lanes <= 64 ? (1 << lsw) == P.slice : (lanes / 64) * (1 << lsw) == P.slice, "chunk %zu: scenarios per wavefront", k);
    std::vector<std::pair<int64_t, int64_t>> use(ng, {0, 0});
    for (int i = 0; i < nrow; ++i) {
      const int32_t* r = rw + 8 * i;
      auto& u = use[i % ng];
      if (u.second == u.first) u = {r[2], r[2] + r[1]};
      CHECK(r[2] == u.first && r[2] + r[1] <= u.second && u.second <= area, "chunk %zu: buffer of row %d", k, r[4]);
      std::vector<Replay::Step> steps;
      std::vector<int> tgt;
      for (int q = r[3]; q < r[8 + 3]; ++q) {
        const int32_t* x = sp + 4 * q;
        const int nu = x[4 + 3] - x[3];
        steps.push_back({x[0], x[1], x[2], nu});
        CHECK(tg + x[3] + nu <= &C.blob[0] + C.ptr[k + 1], "chunk %zu: targets", k);
        for (int j = 0; j < nu; ++j) tgt.push_back(tg[x[3] + j]);
      }
      R.row(r, (int)k, steps, tgt);
    }
    std::sort(use.begin(), use.end());
    for (int i = 1; i < ng; ++i)
      CHECK(use[i].first >= use[i - 1].second || use[i].first == use[i].second, "chunk %zu: buffers overlap", k);
  }
}

int main(int argc, char** argv) {
  if (argc != 5) return 2;
  std::ifstream in(argv[1]);
  int n, m;
  in >> n >> m;
  std::vector<int32_t> bt(n), f(m), t(m), yrp, yci;
  std::vector<double> r(m), x(m), bc(m), g, b;
  for (auto& v : bt) in >> v;
  for (int k = 0; k < m; ++k) in >> f[k] >> t[k] >> r[k] >> x[k] >> bc[k];
  HbmShape shape;
  shape.fp32 = std::strcmp(argv[2], "mixed") == 0;
  shape.batch = std::atoi(argv[3]);
  shape.threads = std::atoi(argv[4]);
  std::string err;
  if (ybus_from_branches(n, m, f.data(), t.data(), r.data(), x.data(), bc.data(), yrp, yci, g, b, err) < 0) return 2;
  Symbolic S;
  if (analyze(n, bt.data(), yrp.data(), yci.data(), g.data(), b.data(), S, err, tail_max_rows(shape.fp32),
              tail_max_level(shape.fp32)) != 0) return 2;
  HbmPlan P;
  if (plan_hbm(S, shape, P, err) != 0) {
    std::printf("refused: %s\n", err.c_str());
    return 3;
  }
  const size_t tsz = shape.fp32 ? 4 : 8, prefix = 4 * (size_t)S.tail_prog_prefix;
  const int waves = shape.threads / 64;
  CHECK(P.chunks.max_ints <= P.chunk_ints, "level chunks beyond the metadata area");
  CHECK(!P.tail_prog_lds || (int)S.tail_prog.size() - S.tail_prog_prefix <= P.chunk_ints, "tail program beyond the metadata area");
  CHECK(P.tail_off % 16 == 0 && P.tail_off >= kScratchBytes + 4 * (size_t)P.chunk_ints + prefix, "row buffers overlap");
  CHECK(P.area >= tail_copy_bytes(S, P.slice, shape.fp32), "the tail copy does not fit");
  const size_t end = P.tail_off + P.area;
  // no more LDS than the schedule takes
  const int counts = (int)P.flow.per_level.size() ? (S.n_fs_levels + 2 + 3) / 4 * 4 : 0;
  const int solve_ints = std::max(P.chunks.max_ints, P.tail_prog_lds ? ((int)S.tail_prog.size() - S.tail_prog_prefix + 3) / 4 * 4 : 0);
  CHECK(P.chunk_ints == std::max({solve_ints, P.row_chunks.max_ints, counts + P.flow_waves * P.flow.max_ints}), "%d words of metadata area", P.chunk_ints);
  CHECK(P.area == std::max({tail_copy_bytes(S, P.slice, shape.fp32), (size_t)P.row_chunks.max_buffer * 4 * tsz * P.slice, (size_t)P.flow_waves * P.flow.max_buffer * 4 * tsz}), "%zu bytes of row buffers", P.area);
  CHECK(P.y_bytes == 0 ? P.y_off == 0 : P.y_off % 16 == 0 && P.y_off >= end && P.y_bytes >= 2 * (size_t)S.nb * P.slice * tsz, "y");
  CHECK(P.lds_bytes >= std::max(end, P.y_off + P.y_bytes) && P.lds_bytes <= shape.max_lds, "%zu bytes of LDS", P.lds_bytes);
  const bool rows = P.factor != FACTOR_LEVELS;
  const char* path = rows ? P.slice == 1 ? "tasks" : "rows" : "levels";
  CHECK((P.factor == FACTOR_LONG_ROWS) == (P.flow.max_ints > kFlowMaxWords), "long records: %d words", P.flow.max_ints);
  if (rows) {
    Replay R(S, P.st);
    if (P.slice == 1) {
      CHECK(P.flow_waves >= 1 && P.flow_waves <= waves, "%d wavefronts take tasks", P.flow_waves);
      CHECK((size_t)P.flow_waves * P.flow_buf * 4 * tsz <= P.area, "row buffers beyond their area");
      replay_tasks(R, P, P.flow_waves);
    } else {
      replay_rows(R, P, shape.threads, tsz);
    }
    R.finish();
  } else {
    CHECK(!P.chunks.f_ptr.empty(), "no factor tasks");
  }
  std::printf("path %s slice %d y %zu lds %zu tail %d longest %d words %d waves %d violations %d\n", path, P.slice, P.y_bytes,
              P.lds_bytes, S.tail_t, S.max_row_blocks, P.flow.max_ints, P.flow_waves, g_fail);
  return g_fail ? 1 : 0;
}
