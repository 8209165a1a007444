// Value refresh of the Jacobian operators (Algorithm 1 for the entry values,
// the block-aware indexing of Algorithm 2 for their placement), fused: one
// thread per (scenario, value of the operator) evaluates the base entry that
// feeds the value at the scenario's state and writes it in the operator's
// value order, so the writes are coalesced for transposed operators too and
// no base value buffer is materialised.  The per-bus state that the entries
// read (voltage and calculated current) is formed once per workgroup in LDS;
// networks too large for that form it in device memory in a launch of its own.
#include "pf_operators.h"

#include <algorithm>

#include "operators.h"

namespace sable {

__global__ void __launch_bounds__(256) k_operator_state(OpParams p) {
#pragma clang fp contract(off)
  const size_t o = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (o >= (size_t)p.count * p.n_bus) return;
  const size_t row = o - o % p.n_bus;
  const int i = (int)(o - row);
  double sn, cs;
  sincos(p.va[o], &sn, &cs);
  const double e = p.vm[o] * cs, f = p.vm[o] * sn;
  double ir = 0.0, ii = 0.0;   // I_i = sum_k Y_ik V_k
  for (int k = p.y_rp[i]; k < p.y_rp[i + 1]; ++k) {
    const size_t c = row + p.y_ci[k];
    double sk, ck;
    sincos(p.va[c], &sk, &ck);
    const double ek = p.vm[c] * ck, fk = p.vm[c] * sk;
    ir += fma(p.y_g[k], ek, -(p.y_b[k] * fk));
    ii += fma(p.y_g[k], fk, p.y_b[k] * ek);
  }
  double4 w;
  w.x = e;
  w.y = f;
  w.z = fma(f, ii, e * ir);      // P_i
  w.w = fma(f, ir, -(e * ii));   // Q_i
  reinterpret_cast<double4*>(p.ef)[o] = w;
}

// F = spec - calc, so every voltage entry is minus the derivative of the
// calculated injection P_i + jQ_i = V_i conj(sum_k Y_ik V_k) (the polar forms
// that Algorithm 1 evaluates, in rectangular products):
//   off the diagonal, with c = V_i V_j cos(theta_ij) = e_i e_j + f_i f_j and
//   s = V_i V_j sin(theta_ij) = f_i e_j - e_i f_j,
//     dP_i/dtheta_j = G s - B c,          dP_i/d|V|_j = (G c + B s) / |V|_j,
//     dQ_i/dtheta_j = -(G c + B s),       dQ_i/d|V|_j = (G s - B c) / |V|_j;
//   on the diagonal, with the row's own P_i and Q_i,
//     dP_i/dtheta_i = -Q_i - B_ii |V_i|^2, dP_i/d|V|_i = P_i / |V|_i + G_ii |V|_i,
//     dQ_i/dtheta_i = P_i - G_ii |V_i|^2,  dQ_i/d|V|_i = Q_i / |V|_i - B_ii |V|_i.
// The value of one entry, by the same operations on every path (the fused ones
// written out), so that neither rounding nor zero, infinite or NaN magnitudes
// depend on where the state is held: bus i (ei, fi, Pi, Qi), bus j (ej, fj)
// and |V| of bus j
__device__ __forceinline__ double entry_value(int kind, bool diag, double G, double B, double2 vi, double2 si,
                                              double2 vj, double magj) {
#pragma clang fp contract(off)
  const bool dva = kind == BK_DP_DVA || kind == BK_DQ_DVA, dp = kind == BK_DP_DVM || kind == BK_DP_DVA;
  double x;
  if (!diag) {
    const double c = fma(vi.x, vj.x, vi.y * vj.y), s = fma(vi.y, vj.x, -(vi.x * vj.y));
    const double gs_bc = fma(G, s, -(B * c)), gc_bs = fma(G, c, B * s);
    if (dva) x = dp ? gs_bc : -gc_bs;
    else x = (dp ? gc_bs : gs_bc) / magj;
  } else {
    if (dva) x = dp ? fma(-magj, B * magj, -si.y) : fma(-magj, G * magj, si.x);
    else x = dp ? fma(G, magj, si.x / magj) : fma(-B, magj, si.y / magj);
  }
  return -x;
}

// thread = (value of the operator, group of kOpGroup scenarios): the
// pattern-side loads (source map, base entry, Y_bus value) once per group
constexpr int kOpGroup = 8;

__global__ void __launch_bounds__(256) k_operator_values(OpParams p) {
  const size_t o = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t groups = ((size_t)p.count + kOpGroup - 1) / kOpGroup;
  if (o >= groups * p.nnz) return;
  const size_t g = o / p.nnz;
  const int v = (int)(o - g * p.nnz);
  const int4 be = p.rec[v];
  const int kind = be.x, i = be.y, j = be.z, q = be.w;
  const double G = (kind != BK_SEL && q >= 0) ? p.y_g[q] : 0.0;
  const double Bv = (kind != BK_SEL && q >= 0) ? p.y_b[q] : 0.0;
  const size_t b1 = min((size_t)p.count, (g + 1) * kOpGroup);
  for (size_t b = g * kOpGroup; b < b1; ++b) {
    double x = 1.0;
    if (kind != BK_SEL) {
      const double4* st = reinterpret_cast<const double4*>(p.ef) + b * p.n_bus;
      const double4 si = st[i];
      double2 vj = make_double2(0.0, 0.0);
      if (i != j) vj = *reinterpret_cast<const double2*>(st + j);
      const double magj = p.vm[b * p.n_bus + j];
      x = entry_value(kind, i == j, G, Bv, make_double2(si.x, si.y), make_double2(si.z, si.w), vj, magj);
    }
    p.values[b * p.nnz + v] = x;
  }
}

// The same with the state in LDS.  A workgroup owns SC scenarios and one of
// `splits` runs of the operator's values: it forms the voltage, |V| and the
// injection of every bus there, then evaluates its values from LDS alone, so
// that the random gathers of a bus pair cost LDS cycles instead of cache lines.
// Bound: the write of the values (8 bytes each), behind 32 bytes of pattern
// per value (record and Y_bus entry) from L2, shared by the SC scenarios.
// J1, J1^T, J2^T and J3^T of 1024 scenarios of the 1354-bus grid (308 MB of
// values, 65 us at the rate of a large copy): 493 us with the state in device
// memory (two launches per operator), 218 us here with two scenarios per
// workgroup.  (Division-free forms of the d/d|V| entries took 201 us, but
// rounded differently and gave values where |V| = 0 has none.)
// OWN: where a scenario's values are split over several workgroups, each would
// form the injections of all buses for the few diagonal entries it has, all of
// them one after the other in front of its values (3900 buses, one scenario: 73
// us for the four operators, 67 by the two-launch path); there a diagonal entry
// forms its own bus's (49 us).
constexpr int kOpBusDoubles = 5;   // (e, f), (P, Q), |V|

template <int SC, bool OWN>
__global__ void __launch_bounds__(1024) k_operator_lds(OpParams p, int splits) {
#pragma clang fp contract(off)
  extern __shared__ __align__(16) double op_smem[];
  const int n = p.n_bus, tid = threadIdx.x, nt = blockDim.x;
  double2* v2 = reinterpret_cast<double2*>(op_smem);       // [n][SC]
  double2* pq = v2 + (size_t)n * SC;                       // [n][SC]
  double* mag = reinterpret_cast<double*>(pq + (size_t)n * SC);
  const int group = blockIdx.x / splits, split = blockIdx.x - group * splits;
  const int b0 = group * SC;
  for (int q = tid; q < n * SC; q += nt) {
    const int s = q / n, i = q - s * n;
    double sn = 0.0, cs = 1.0, v = 1.0;
    if (b0 + s < p.count) {
      const size_t o = (size_t)(b0 + s) * n + i;
      sincos(p.va[o], &sn, &cs);
      v = p.vm[o];
    }
    v2[i * SC + s] = make_double2(v * cs, v * sn);
    mag[i * SC + s] = v;
  }
  __syncthreads();
  auto injection = [&](int i, double2 (&out)[SC]) {   // (P, Q) of bus i
    double ir[SC], ii[SC];
#pragma unroll
    for (int s = 0; s < SC; ++s) ir[s] = ii[s] = 0.0;
    for (int k = p.y_rp[i]; k < p.y_rp[i + 1]; ++k) {
      const int j = p.y_ci[k];
      const double g = p.y_g[k], b = p.y_b[k];
#pragma unroll
      for (int s = 0; s < SC; ++s) {
        const double2 w = v2[j * SC + s];
        ir[s] += fma(g, w.x, -(b * w.y));
        ii[s] += fma(g, w.y, b * w.x);
      }
    }
#pragma unroll
    for (int s = 0; s < SC; ++s) {
      const double2 w = v2[i * SC + s];
      out[s] = make_double2(fma(w.y, ii[s], w.x * ir[s]), fma(w.y, ir[s], -(w.x * ii[s])));
    }
  };
  if (!OWN) {
    for (int i = tid; i < n; i += nt) {
      double2 x[SC];
      injection(i, x);
#pragma unroll
      for (int s = 0; s < SC; ++s) pq[i * SC + s] = x[s];
    }
    __syncthreads();
  }
  const int per = (p.nnz + splits - 1) / splits;
  const int v1 = min(p.nnz, (split + 1) * per);
  for (int v = split * per + tid; v < v1; v += nt) {
    const int4 r = p.rec[v];
    const int kind = r.x, i = r.y, j = r.z;
    const bool sel = kind == BK_SEL, y = !sel && r.w >= 0;
    const double G = y ? p.y_g[r.w] : 0.0, B = y ? p.y_b[r.w] : 0.0;
    double2 own[SC] = {};
    if (OWN && i == j && !sel) injection(i, own);
#pragma unroll
    for (int s = 0; s < SC; ++s) {
      if (b0 + s >= p.count) break;
      if (!OWN) own[s] = pq[i * SC + s];
      const double x = entry_value(kind, i == j, G, B, v2[i * SC + s], own[s], v2[j * SC + s], mag[j * SC + s]);
      p.values[(size_t)(b0 + s) * p.nnz + v] = sel ? 1.0 : x;
    }
  }
}

constexpr size_t kOpLdsLimit = 160 * 1024;

bool operator_state_in_lds(int n_bus) {
  return (size_t)n_bus * kOpBusDoubles * sizeof(double) <= kOpLdsLimit;
}

hipError_t set_operator_lds(int n_bus) {
  if (2 * (size_t)n_bus * kOpBusDoubles * sizeof(double) <= 64 * 1024) return hipSuccess;   // the default limit
  hipError_t e = hipSuccess;
  for (const void* f : {reinterpret_cast<const void*>(&k_operator_lds<1, false>),
                        reinterpret_cast<const void*>(&k_operator_lds<1, true>),
                        reinterpret_cast<const void*>(&k_operator_lds<2, false>)}) {
    const hipError_t r = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kOpLdsLimit);
    if (r != hipSuccess) e = r;
  }
  return e;
}

hipError_t launch_operator_values(const OpParams& p, hipStream_t st) {
  const size_t nst = (size_t)p.count * p.n_bus, total = (size_t)p.count * p.nnz;
  if (total == 0) return hipSuccess;
  if (operator_state_in_lds(p.n_bus)) {
    // two scenarios per workgroup where that still leaves one per compute
    // unit, and the values of few scenarios split over as many workgroups as
    // there are compute units.  Threads: at least one and a half per bus, as a
    // power of two from a wavefront to 512, and 1024 from 512 buses on.  The four operators of 14 buses x60000 took
    // 454 us with 512 threads, most of them idle, against 166 with 64 (two
    // launches: 222); 30 buses x40000 359 and 164; 60 x20000 237 and 152 (128);
    // 118 x11000 184 and 159 (256), where 64 take 217; 300 x4000 154 with 512,
    // 169 with 256; 1354 x1024 (one set of buffers) 234 with 512, 177 with 1024
    constexpr int kCus = 256;
    const size_t bus = kOpBusDoubles * sizeof(double) * (size_t)p.n_bus;
    const int sc = p.count >= 2 * kCus && 2 * bus <= kOpLdsLimit ? 2 : 1;
    int nt = p.n_bus >= 512 ? 1024 : 64;
    while (nt < 512 && 2 * nt < 3 * p.n_bus) nt *= 2;
    const int groups = (p.count + sc - 1) / sc;
    const int splits = std::max(1, std::min((p.nnz + nt - 1) / nt, kCus / groups));
    // each diagonal entry forms its bus's injection from four splits on (3900
    // buses x64, four splits: 118 us against 126; x120, two: 192 against 160)
    const bool own = splits >= 4;
    const dim3 g((unsigned)((size_t)groups * splits)), b(nt);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, g, b, sc * bus, st, p, splits); };
    if (sc == 2) launch(k_operator_lds<2, false>);
    else if (own) launch(k_operator_lds<1, true>);
    else launch(k_operator_lds<1, false>);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_operator_state, dim3((unsigned)((nst + 255) / 256)), dim3(256), 0, st, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const size_t work = ((size_t)p.count + kOpGroup - 1) / kOpGroup * p.nnz;
  hipLaunchKernelGGL(k_operator_values, dim3((unsigned)((work + 255) / 256)), dim3(256), 0, st, p);
  return hipGetLastError();
}

// Block-diagonal embedding of one scenario's CSR pattern (eq. BDE_global):
// scenario b's block sits at row offset b * rows and column offset b * cols,
// its values at offset b * nnz.  One thread per global row pointer and per
// global column index.
__global__ void __launch_bounds__(256) k_bde_csr(const int* indptr, const int* indices, int rows, int cols,
                                                 int nnz, int count, int64_t* crow, int64_t* col) {
  const size_t o = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t nr = (size_t)count * rows, nc = (size_t)count * nnz;
  if (o <= nr) {
    const size_t b = rows > 0 ? o / rows : 0, r = o - b * rows;
    crow[o] = (o == nr) ? (int64_t)nc : (int64_t)b * nnz + indptr[r];
  }
  if (o < nc) {
    const size_t b = o / nnz, v = o - b * nnz;
    col[o] = (int64_t)b * cols + indices[v];
  }
}

hipError_t launch_bde_csr(const int* indptr, const int* indices, int rows, int cols, int nnz, int count,
                          int64_t* crow, int64_t* col, hipStream_t st) {
  const size_t work = std::max((size_t)count * rows + 1, (size_t)count * nnz);
  hipLaunchKernelGGL(k_bde_csr, dim3((unsigned)((work + 255) / 256)), dim3(256), 0, st, indptr, indices, rows,
                     cols, nnz, count, crow, col);
  return hipGetLastError();
}

}  // namespace sable

