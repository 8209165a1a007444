// Launch plan of HBM-resident templates (declared in hbm_plan.h).
#include "hbm_plan.h"

#include <algorithm>

#include "sable_pf.h"

namespace sable {

namespace {

// least metadata budget (int32 words)
constexpr int32_t kMinChunkInts = 2048;

// LDS before the row buffers / the tail copy besides the metadata: the kernels'
// scratch and the tail program's solve prefix
size_t fixed_bytes(const Symbolic& S) { return kScratchBytes + (4 * (size_t)S.tail_prog_prefix + 15) / 16 * 16; }

// the plan for slices of p.slice scenarios that factor row by row (rows) or by
// levels in place, with y in LDS where that leaves the full metadata budget (if
// want_y); waves: wavefronts that take tasks (rows of one scenario)
int plan_slice(const Symbolic& S, const HbmShape& h, bool rows, bool want_y, int waves, HbmPlan& p,
               std::string& err) {
  const int sl = p.slice;
  const size_t tsz = h.fp32 ? 4 : 8;
  const size_t upd_words = S.tail_prog.size() - (size_t)S.tail_prog_prefix;
  const size_t fixed = fixed_bytes(S);
  const size_t tail_bytes = tail_copy_bytes(S, sl, h.fp32);
  // what the metadata can have beside the tail copy (S > 1: at most half of it
  // where rows need buffers) and, when that leaves the full metadata budget,
  // beside y: every solve's gathers then stay on chip
  if (fixed + tail_bytes + 4 * kMinChunkInts > h.max_lds) {
    err = "pf_template_build: the dense tail does not fit in LDS";
    return PF_EINVAL;
  }
  size_t room = h.max_lds - fixed - tail_bytes;
  p.y_bytes = want_y ? ((size_t)2 * S.nb * sl * tsz + 15) / 16 * 16 : 0;
  const int32_t want = rows && sl > 1 ? kChunkInts / 2 : kChunkInts;
  if (room >= p.y_bytes + 4 * (size_t)want) room -= p.y_bytes;
  else p.y_bytes = 0;
  const int32_t budget = (int32_t)std::min<size_t>(want, room / 16 * 4);
  p.st = rows ? storage_split(S) : storage_by_position(S);
  int rc = build_level_chunks(S, budget, p.chunks, err, &p.st);
  if (rc != 0) return rc;
  // the tail's update words are staged in the metadata area (free while the
  // tail is factored) when the area, grown within the room, holds them
  p.tail_prog_lds = (upd_words + 3) / 4 * 16 <= room;
  const int solve_ints = std::max<int>(p.chunks.max_ints, p.tail_prog_lds ? (int)(upd_words + 3) / 4 * 4 : 0);
  p.chunk_ints = solve_ints;
  p.row_chunks = RowChunks{};
  p.flow = FlowTasks{};
  p.area = tail_bytes;
  p.factor = rows ? FACTOR_ROWS : FACTOR_LEVELS;
  if (rows) {
    p.chunk_ints = std::max(p.chunk_ints, budget);
    const int counts = (S.n_fs_levels + 2 + 3) / 4 * 4;   // wavefront tasks: the levels' counts and the next task
    if (sl == 1) {
      // each wavefront has its share of the metadata area and of the buffers.
      // A long row's record takes more than that, out of what the buffers would have.
      p.flow_waves = waves;
      p.flow_meta = std::min<int>(kFlowMaxWords, std::max(0, p.chunk_ints - counts) / waves / 4 * 4);
      p.flow_meta = std::max(p.flow_meta, flow_row_words(S));
      p.chunk_ints = std::max(p.chunk_ints, counts + waves * p.flow_meta);
    }
    if (fixed + p.y_bytes + 4 * (size_t)p.chunk_ints + tail_bytes > h.max_lds) {
      err = "pf_template_build: the task records do not fit in LDS";
      return PF_EINVAL;
    }
    p.area = h.max_lds - fixed - p.y_bytes - 4 * (size_t)p.chunk_ints;
    if (sl == 1) {
      p.flow_buf = (int)(p.area / (4 * tsz)) / waves;
      rc = build_flow_tasks(S, p.st, waves, p.flow_buf, p.flow_meta, p.flow, err);
      if (p.flow.max_ints > kFlowMaxWords) p.factor = FACTOR_LONG_ROWS;
    } else {
      rc = build_row_chunks(S, p.st, sl, h.threads, (int64_t)(p.area / (4 * tsz * sl)), budget, p.row_chunks, err);
    }
    if (rc != 0) return rc;
    // and no more of it than the schedule takes, so that several of the smaller
    // workgroups that block_threads selects share a compute unit (300 buses x1000,
    // FP64, 128 threads: 0.70 ms with 39 KB per workgroup, 1.08 with all 160; with
    // 1024 threads the registers leave room for one)
    if (sl == 1) {
      p.flow_meta = p.flow.max_ints;
      p.flow_buf = p.flow.max_buffer;
      p.chunk_ints = std::max(solve_ints, counts + waves * p.flow_meta);
      p.area = std::max(tail_bytes, (size_t)waves * p.flow_buf * 4 * tsz);
    } else {
      p.chunk_ints = std::max(solve_ints, p.row_chunks.max_ints);
      p.area = std::max(tail_bytes, (size_t)p.row_chunks.max_buffer * 4 * tsz * sl);
    }
  }
  p.tail_off = fixed + 4 * (size_t)p.chunk_ints;
  p.lds_bytes = (p.tail_off + p.area + 15) / 16 * 16;
  p.y_off = p.y_bytes ? p.lds_bytes : 0;
  p.lds_bytes += p.y_bytes;
  return 0;
}

// the elimination steps that follow one another: row by row, the most of a row
// in each level; by levels, the most that a row takes in each of them
struct Chains { int64_t rows = 0, levels = 0; };
Chains step_chains(const Symbolic& S) {
  Chains c;
  auto steps = [&](int32_t a) { return (a < S.tail_base ? S.diag[a] : S.tail_split[a - S.tail_base]) - S.rp[a]; };
  for (int32_t h = 0; h < S.n_fs_levels; ++h) {
    int32_t most = 0;
    for (int32_t q = S.lev_l_ptr[h]; q < S.lev_l_ptr[h + 1]; ++q) most = std::max(most, steps(S.lev_l_rows[q]));
    c.rows += most;
  }
  int32_t tail = 0;
  for (int32_t a = S.tail_base; a < S.nb; ++a) tail = std::max(tail, steps(a));
  c.rows += tail;
  for (int32_t h = 0; h < S.n_task_levels; ++h) {
    int32_t most = 0;
    for (int32_t i = S.task_ptr[h]; i < S.task_ptr[h + 1]; ++i)
      most = std::max(most, S.task4[4 * (size_t)i + 2] - S.task4[4 * (size_t)i + 1]);
    c.levels += most;
  }
  return c;
}

// Whether slices of this many scenarios rather factor row by row than by levels.
// The rows move fewer bytes, the levels have more lanes at work and wait less on
// one step after the other (solves below in ms, by rows / by levels, with 1024
// threads and the batches that give this width).
bool prefer_rows(const Symbolic& S, const HbmShape& h, int slice) {
  const size_t tsz = h.fp32 ? 4 : 8;
  if (slice > 1) {
    // Networks of a few buses, which only block_threads brings here, by levels:
    // nearly all their rows are in the tail (with the adjoint, FP32: 14 buses x600,
    // 256 threads 0.244 / 0.226, x4096, 1024 threads 0.301 / 0.286; 30 x4096 0.387 /
    // 0.372).
    if (S.nb < 48) return false;
    // Rows where one value of all scenarios of a block is a run of 64 bytes or
    // more (FP64, eight: 300 buses 1.13 / 1.17, 1354 6.29 / 8.03; FP32, sixteen:
    // 300 2.44 / 2.46) ...
    if (slice * tsz >= 64) return true;
    // ... or where a few long rows make the levels as serial (FP64, two: a hub of
    // 400 leaves 0.98 / 1.40, two of 200 1.06 / 1.12) ...
    const Chains c = step_chains(S);
    const double serial = double(c.rows) - 2.0 * c.levels;   // a step of a level takes about two of a row
    if (c.rows >= 128 && 8 * serial <= c.rows) return true;
    // ... else where the factors of one slice per compute unit leave the 256 MB
    // Infinity Cache (with the rest of the state, from about 175 MB on), and are
    // large against the rows' chain of steps.  FP64, two: 1354 buses (138 MB) 3.00 /
    // 2.72, 2600 (0.63 MB per step) 4.33 / 4.49, 1200 of three branches each
    // (0.16) 7.75 / 6.42; four: 700 (147 MB) 1.36 / 1.32, 1354 (1.2) 4.59 / 4.68,
    // the 1200 (0.32) 10.4 / 10.1, 2000 of two branches (0.51) 8.66 / 9.00.  FP32,
    // four: 1354 (138 MB) 5.72 / 5.42, 2600 (1.1) 8.08 / 8.80, the 2000 (0.39) 9.46 /
    // 9.30; eight: 700 (147 MB) 3.24 / 3.12, 1000 (183 MB) 3.74 / 3.90, the 1200
    // (0.51) 13.6 / 13.9.
    const double mb = 1e-6 * h.n_cu * slice * S.nnzb() * 4 * tsz;
    return mb >= 175 && mb >= 0.5 * serial;
  }
  // One scenario: as tasks, which need many wavefronts to overlap the levels.
  // From twelve on FP64 always (x250: 300 buses 0.285 / 0.312, 1354 0.985 / 1.00,
  // 4000 2.08 / 2.53), FP32 on the larger grids (x250: 1354 1.63 / 1.56, 2800
  // 2.37 / 2.34, 3400 2.44 / 2.50, 9241 8.75 / 9.45).  A compute unit holds two
  // or more of the narrower workgroups by levels, fewer with the row buffers:
  // eight wavefronts, FP64 x250: 1354 1.17 / 1.06, 2600 1.47 / 1.47, 4000 2.35 /
  // 2.64, FP32: 4000 3.53 / 3.45, 9241 10.7 / 11.1; four, FP64: 1354 1.77 / 1.38,
  // 9241 x250 12.4 / 13.4, x500 24.8 / 21.1; one, 9241 x250: 38.2 / 35.6.
  if (h.threads >= 768) return !h.fp32 || S.nb >= 3072;
  if (h.threads >= 512) return S.nb >= (h.fp32 ? 4096 : 2560);
  return h.threads >= 256 && S.nb >= 4096 && h.batch <= h.n_cu;
}

}  // namespace

int plan_hbm(const Symbolic& S, const HbmShape& h, HbmPlan& p, std::string& err) {
  // S scenarios interleaved per slice, S as large as keeps at least one slice
  // per compute unit and leaves room in LDS for the tail copy and for staged
  // metadata; S = 1 always fits: the tail holds at most 32 x 32 blocks.  The
  // rows of the row-by-row factorisation have to fit beside the metadata too
  // (in the place of the tail copy, which is made after it).  Where they do not,
  // y gives way to them, and with S = 1 some of the wavefronts that take tasks.
  // With FP32 factors neither does: the refinement solves, which y in LDS is for,
  // are the larger part (11000 buses, mixed: x250 9.8 ms by levels, 10.2 by tasks
  // without y, 9.8 by half as many wavefronts, x37 7.0 and 8.1; FP64 x250 10.6
  // by levels, 6.8 by tasks without y).
  // Rows that are too long for S scenarios may still fit half as many; beyond
  // that the slice keeps its width and factors by levels in place (FP64 x4200, a
  // hub of 400 leaves: 2.27 ms by levels of 16 scenarios, 1.92 by rows of 8, 2.62
  // of 4; of 1000 leaves: 6.4 and, by rows of 2, 10.3; of 2000 leaves by levels of
  // 16 and of one scenario: 18.9 and 75).  Only FP64 slices of two go to one: the
  // width that tests/test_gpu_rows.py pins for a star of 2000 leaves x520,
  // although two by levels would be faster (x600: 10.4 against 13.0 ms).
  p = HbmPlan{};
  while (p.slice < kMaxSlice && h.batch / (2 * p.slice) >= h.n_cu) p.slice *= 2;
  while (p.slice > 1 && fixed_bytes(S) + tail_copy_bytes(S, p.slice, h.fp32) + 4 * kMinChunkInts > h.max_lds) p.slice /= 2;
  const int width = p.slice;
  auto rows_fit = [&](int slice) {
    p.slice = slice;
    int waves = h.threads / 64;
    if (plan_slice(S, h, true, true, waves, p, err) == 0) return true;
    if (h.fp32) return false;
    if (plan_slice(S, h, true, false, waves, p, err) == 0) return true;
    while (slice == 1 && waves > 1)
      if (plan_slice(S, h, true, false, waves /= 2, p, err) == 0) return true;
    return false;
  };
  const bool rows = prefer_rows(S, h, width);
  if (rows && (rows_fit(width) || (width > 2 && rows_fit(width / 2)))) return 0;
  for (p.slice = rows && width == 2 && !h.fp32 ? 1 : width; p.slice >= 1; p.slice /= 2)
    if (plan_slice(S, h, false, true, 0, p, err) == 0) return 0;
  return PF_EINVAL;
}

}  // namespace sable
