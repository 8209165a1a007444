// Launch plan of HBM-resident templates (host only): how many scenarios a slice
// interleaves, how it factors, and what of a workgroup's LDS each part gets.
//
// LDS of a workgroup, in this order: the kernels' scratch, the metadata area
// (level chunks; row chunks, or the records and counts of the wavefront tasks),
// the tail program's solve prefix, the row buffers of the row-by-row
// factorisation or, after it and in the same place, the copy of the dense tail,
// and y, the solves' right-hand side / solution vector, where it fits.
#pragma once

#include <cstddef>
#include <cstdint>
#include <string>

#include "symbolic.h"

namespace sable {

constexpr int kMaxSlice = 16;        // scenarios per workgroup
constexpr int kScratchBytes = 4096;  // LDS scratch at the start of every kernel's dynamic LDS

// largest level-metadata chunk an HBM-resident workgroup stages in LDS
// (int32 words; 48 KB)
constexpr int32_t kChunkInts = 12288;

// The dense tail of an LDS-resident slice lives in registers: at most 32 block
// rows in FP32, 16 in FP64.
constexpr int32_t tail_max_rows(bool fp32) { return fp32 ? 32 : 16; }
// And an FP64 tail takes in levels of at most four rows: a row costs the tail
// 0.7 us per factorisation, a level outside it 2.6 us per update (factor and
// backward pass), which the tail's wavefront alone no longer beats.  So it is in
// HBM-resident templates, though only networks of a few buses have such levels at
// the top (14 buses, block_threads 256, x600: 98 us with the limit, 105 without,
// x4096: 214 and 306; 150 buses x4096: 0.83 and 0.89 ms).  With FP32 factors a
// level also costs the refinement's four solves, a tail row less.
constexpr int32_t tail_max_level(bool fp32) { return fp32 ? tail_max_rows(true) : 4; }

// How a template factors: by levels in place, or row by row (one scenario per
// slice: as wavefront tasks); long rows: with task records beyond kFlowMaxWords.
enum Factoring : int { FACTOR_LEVELS = 0, FACTOR_ROWS = 1, FACTOR_LONG_ROWS = 2 };

struct HbmShape {
  int32_t batch = 1, threads = 1024;
  int32_t n_cu = 256;
  size_t max_lds = 160 * 1024;
  bool fp32 = false;
};

struct HbmPlan {
  int32_t slice = 1;             // scenarios per workgroup
  Factoring factor = FACTOR_LEVELS;
  LuStorage st;
  LevelChunks chunks;
  RowChunks row_chunks;
  FlowTasks flow;
  int32_t chunk_ints = 0;        // words of the metadata area
  bool tail_prog_lds = false;    // the tail program's update words are staged there
  int32_t flow_waves = 0;        // wavefronts that take tasks
  int32_t flow_buf = 0;          // row buffer of a wavefront, in blocks
  int32_t flow_meta = 0;         // words of a wavefront's task record area
  size_t tail_off = 0;           // byte offset of the row buffers / the tail copy
  size_t area = 0;               // bytes there
  size_t y_off = 0, y_bytes = 0; // y (0: in device memory)
  size_t lds_bytes = 0;
};

// stride of a scenario's blocks in the LDS copy of the tail: odd, so that the
// scenarios' copies start in different banks
inline size_t tail_copy_stride(const Symbolic& S) { return S.tail_cblk.size() | 1; }
// bytes of the copy: per scenario the tail-column blocks, pivot inverses and
// right-hand sides
inline size_t tail_copy_bytes(const Symbolic& S, int slice, bool fp32) {
  return (size_t)slice * (fp32 ? 4 : 8) * (4 * tail_copy_stride(S) + 6 * (size_t)S.tail_t);
}

// Returns 0, or PF_EINVAL (err set) when the network does not fit.
int plan_hbm(const Symbolic& S, const HbmShape& shape, HbmPlan& out, std::string& err);

}  // namespace sable
