// Wide-batch operator products on the matrix cores (gfx950).
//
// With 8 or more right-hand sides the CSR row products of the CG iteration are
// bound by their vector gathers: every nonzero fetches a whole ld-wide slice
// of the vector it multiplies, so at 32 columns the gathers move about 30
// times the bytes of the matrix.  Here the coupling matrices are stored by
// blocks of 16 rows: the columns that any row of a block uses, sixteen at a
// time, as dense units of 16 rows x 16 listed columns (four k-steps of the
// 16x16x4 matrix instructions).  A row of the multiplied vector is one
// contiguous ld-wide segment wherever it lies, and the instruction's four
// column slots are loaded by different lanes, so the listed columns need not
// be neighbours: a unit's vector rows are gathered at no extra cost, each
// fetched once per block instead of once per nonzero.  Naming single columns
// instead of blocks of them leaves fewer stored zeros: on the peridynamic
// interface rows (h = 1/160) 73 % of the values are nonzero, against 62 % with
// aligned blocks of 8 columns, 54 % with 16, and 63 % with single columns over
// 32-row blocks.
//
// The interior solves w = K_II^-1 y, a dense product per subdomain, use the
// same instruction on 16x16 tiles of the explicit inverse (FP64), or
// v_mfma_f32_16x16x4f32 with FP32 accumulation in the mixed path.
//
// Operator of the CG iteration these kernels serve: S p summed over
// subdomains (eq. subSchurComplement, summed as in eq. SchurComplement),
// y = K_IG z, w = K_II^-1 y + beta w_before (= K_II^-1 K_IG p), q = K_GG p - K_GI w.
//
// Per output column the arithmetic depends only on that column (the matrix
// instructions compute each output element from its own row and column), so
// a column's result does not depend on the batch width among the widths this
// path serves; it differs in rounding from the CSR kernels of narrow batches.
#pragma once
#include <type_traits>

#include "dd_kernels.h"

namespace dd {

constexpr int kT = 16;   // tile edge

// Tile storage: 256 values per tile; lane l of the wave holds
// T[l % 16][4 s + l / 16], the A operand of step s (s = 0..3) of the 16x16x4
// instruction.  FP64 tiles keep steps 0-1 of lane l at 2l, 2l+1 and steps 2-3
// at 128 + 2l, 128 + 2l + 1, so that each of a wave's two 16-byte loads reads
// 1 KB contiguous (whole cache lines); FP32 tiles keep the four steps of lane
// l at 4l .. 4l+3, one 16-byte load per lane.
template <typename T> struct TileLayout;
template <> struct TileLayout<double> {
  static __host__ __device__ constexpr int pos(int l, int s) { return (s >> 1) * 128 + 2 * l + (s & 1); }
  static __host__ __device__ constexpr int lane(int p) { return (p & 127) >> 1; }
  static __host__ __device__ constexpr int step(int p) { return ((p >> 7) << 1) | (p & 1); }
};
template <> struct TileLayout<float> {
  static __host__ __device__ constexpr int pos(int l, int s) { return 4 * l + s; }
  static __host__ __device__ constexpr int lane(int p) { return p >> 2; }
  static __host__ __device__ constexpr int step(int p) { return p & 3; }
};

// Coupling units: 16 rows x 16 listed columns in the tile order above; unit t
// lists its columns at tcol[t].[g], the four of lane group g = lane / 16 (its
// A operands' columns in step order), as one int4.
constexpr int kUV = kT * kT;
// Place in a block's column lists of its t-th column (in increasing order):
// column kk = t % 16 of unit t / 16 is step kk / 4 of lane group kk % 4.
__host__ __device__ constexpr int unit_slot(int t) { return t / kT * kT + t % 4 * 4 + t % kT / 4; }

// Values of a CSR matrix into its (zeroed) FP64 units, one workgroup per row
// block, 16 lanes per row: a lane finds its entries' columns in the block's list
// (units [tptr, tsplit) hold the entries [ptr, split), units [tsplit, tptr + 1) the
// others; split and tsplit may be nullptr).  A row that repeats a column (or
// lists its columns out of order) is left to one lane, which adds its entries
// in order.  Bound: the latency of the searches, in LDS where the list fits
// (one thread per row, searching in memory, took 1.6 ms on the peridynamic
// interface rows, this 0.28 ms).
constexpr int kFillList = 4096;
__global__ void __launch_bounds__(kT * kT)
k_fill_units(int nrows, const int *__restrict__ ptr, const int *__restrict__ split, const int *__restrict__ col,
             const double *__restrict__ val, const int *__restrict__ tptr, const int *__restrict__ tsplit,
             const int *__restrict__ tcol, double *__restrict__ unit) {
  __shared__ int lds[kFillList];
  const int rb = blockIdx.x, ii = threadIdx.x / kT, lane = threadIdx.x % kT, i = rb * kT + ii;
  const int t0 = tptr[rb], t2 = tptr[rb + 1], t1 = tsplit ? tsplit[rb] : t2;
  const bool in_lds = (t2 - t0) * kT <= kFillList;
  if (in_lds)
    for (int k = threadIdx.x; k < (t2 - t0) * kT; k += kT * kT) lds[k] = tcol[(size_t)t0 * kT + unit_slot(k)];
  __syncthreads();
  if (i >= nrows) return;
  const int b = ptr[i], e = ptr[i + 1], mid = split ? split[i] : e;
  auto place = [&](int a) {
    const int u0 = a < mid ? t0 : t1, u1 = a < mid ? t1 : t2, c = col[a];
    int lo = 0, hi = (u1 - u0) * kT - 1;          // first place of c
    while (lo < hi) {
      const int m = (lo + hi) / 2;
      const int cm = in_lds ? lds[(u0 - t0) * kT + m] : tcol[(size_t)u0 * kT + unit_slot(m)];
      if (cm < c) lo = m + 1;
      else hi = m;
    }
    const int kk = lo % kT;
    // U[ii][kk] is held by lane (kk % 4) * 16 + ii at step kk / 4
    unit[((size_t)u0 + lo / kT) * kUV + TileLayout<double>::pos((kk % 4) * kT + ii, kk / 4)] += val[a];
  };
  bool repeats = false;
  for (int a = b + 1 + lane; a < e; a += kT) repeats |= a != mid && col[a] <= col[a - 1];
  for (int o = 1; o < kT; o *= 2) repeats |= __shfl_xor((int)repeats, o) != 0;
  if (!repeats)
    for (int a = b + lane; a < e; a += kT) place(a);
  else if (lane == 0)
    for (int a = b; a < e; ++a) place(a);
}

// FP64 tiles -> the FP32 copies of the mixed path (the same values rounded, in
// the FP32 tile order).
__global__ void k_units_to_f32(size_t nunit, const double *__restrict__ in, float *__restrict__ out) {
  for (size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x; o < nunit * kUV;
       o += (size_t)gridDim.x * blockDim.x) {
    const size_t t = o / kUV;
    const int r = (int)(o - t * kUV);
    out[o] = (float)in[t * kUV + TileLayout<double>::pos(TileLayout<float>::lane(r), TileLayout<float>::step(r))];
  }
}

// Columns of the vector slices: with NCB column blocks of 16 (ld = 16 NCB for
// NCB >= 2) lane l holds the NCB consecutive columns NCB (l % 16) + q, q < NCB,
// of each row it reads, so that one 16- or 32-byte load brings all of them
// (the q-th matrix instruction then computes the columns NCB j + q, j < 16).
// For NCB = 1 lane l holds column l % 16; below ld = 16 the lanes past the last
// column read the columns again (their products land in output columns that
// are not stored).
template <int NCB>
__device__ __forceinline__ int slice_col0(int l16, int ld) {
  return NCB == 1 ? (l16 & (ld - 1)) : NCB * l16;
}
template <int NCB>
__device__ __forceinline__ void slice_row(const double *__restrict__ p, double (&v)[NCB]) {
  if constexpr (NCB == 1) {
    v[0] = p[0];
  } else {
    typedef double vt __attribute__((ext_vector_type(NCB)));
    const vt w = *(const vt *)p;
#pragma unroll
    for (int q = 0; q < NCB; ++q) v[q] = w[q];
  }
}
template <int NCB>
__device__ __forceinline__ void slice_row(const float *__restrict__ p, float (&v)[NCB]) {
  if constexpr (NCB == 1) {
    v[0] = p[0];
  } else {
    typedef float vt __attribute__((ext_vector_type(NCB)));
    const vt w = *(const vt *)p;
#pragma unroll
    for (int q = 0; q < NCB; ++q) v[q] = w[q];
  }
}

// A operand of a streamed coupling unit, FP64 or FP32 (nontemporal loads).
__device__ __forceinline__ void unit_a(const double *unit, int lane, double (&a)[4]) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  const v2 u = __builtin_nontemporal_load((const v2 *)(unit + 2 * lane));
  const v2 v = __builtin_nontemporal_load((const v2 *)(unit + 128 + 2 * lane));
  a[0] = u[0]; a[1] = u[1]; a[2] = v[0]; a[3] = v[1];
}
__device__ __forceinline__ void unit_a(const float *unit, int lane, float (&a)[4]) {
  typedef float v4 __attribute__((ext_vector_type(4)));
  const v4 v = __builtin_nontemporal_load((const v4 *)(unit + 4 * lane));
  a[0] = v[0]; a[1] = v[1]; a[2] = v[2]; a[3] = v[3];
}

// acc[q] += sgn * U * X over the units t0, t0 + st, t0 + 2 st, ... (< t1) of one
// row block, in that order (t0, t1, st uniform over the wave).  FP64 units run
// on v_mfma_f64_16x16x4f64.  FP32 units (mixed path) run on
// v_mfma_f32_16x16x4f32 (twice the rate): the vector is rounded to FP32, two
// steps accumulate 8 products per output element in FP32, and these sums are
// added to the FP64 accumulators, so FP32 rounding enters only within them
// (rows are then in the FP32 instruction's order: row 4 (l / 16) + r of lane l,
// register r).  WIDE: FP32 units and vector rows are widened and run on the FP64
// instruction (every product and sum in FP64; the four-launch iteration, whose CSR
// rows hold them in FP64 too).  A pass of the loop runs unit j while the operands
// of units j + 1 .. j + D - 1 and the column lists of the D after them are in
// flight.  Scheduling barriers keep every group of loads in program
// order, so that the instructions of one buffer wait only for that buffer's
// loads; the loads past a wave's last unit are skipped.
template <int NCB, int D, bool WIDE, typename VT, typename XT>
__device__ __forceinline__ void tile_row_acc(int t0, int t1, int st, const int4 *__restrict__ tcol,
                                             const VT *__restrict__ tval, const XT *__restrict__ x, int ld,
                                             double sgn, dbl4 (&acc)[NCB]) {
  const int cnt = t0 < t1 ? (t1 - t0 + st - 1) / st : 0;
  if (cnt == 0) return;
  const int lane = lane_id(), g = lane >> 4;
  const XT *xc = x + slice_col0<NCB>(lane & 15, ld);
  const int4 *cl = tcol + (size_t)t0 * 4 + g;
  const VT *tv = tval + (size_t)t0 * kUV;
  VT a[D][4];
  XT xs[D][4][NCB];
  int4 ix[D];
  auto list = [&](int d, int j) { ix[d] = cl[(size_t)j * st * 4]; };
  auto load = [&](int d, int j) {
    unit_a(tv + (size_t)j * st * kUV, lane, a[d]);
    slice_row<NCB>(xc + (size_t)ix[d].x * ld, xs[d][0]);
    slice_row<NCB>(xc + (size_t)ix[d].y * ld, xs[d][1]);
    slice_row<NCB>(xc + (size_t)ix[d].z * ld, xs[d][2]);
    slice_row<NCB>(xc + (size_t)ix[d].w * ld, xs[d][3]);
  };
  auto mma = [&](int d) {
    if constexpr (std::is_same<VT, float>::value && !WIDE) {
      const float fs = (float)sgn;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        flt4 c[NCB];
#pragma unroll
        for (int q = 0; q < NCB; ++q) {
          const flt4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
          c[q] = mfma16x16x4(a[d][2 * h], fs * (float)xs[d][2 * h][q], zero);
          c[q] = mfma16x16x4(a[d][2 * h + 1], fs * (float)xs[d][2 * h + 1][q], c[q]);
        }
#pragma unroll
        for (int q = 0; q < NCB; ++q)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[q][r] += (double)c[q][r];
      }
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int q = 0; q < NCB; ++q) acc[q] = mfma16x16x4((double)a[d][s], sgn * (double)xs[d][s][q], acc[q]);
    }
  };
  // (list and operand buffers are filled past the end with the last unit's)
#pragma unroll
  for (int d = 0; d < D; ++d) list(d, min(d, cnt - 1));
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int d = 0; d < D; ++d) {
    load(d, min(d, cnt - 1));
    list(d, min(d + D, cnt - 1));
    __builtin_amdgcn_sched_barrier(0);
  }
  int j = 0;
  for (; j + 2 * D <= cnt; j += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      mma(d);
      __builtin_amdgcn_sched_barrier(0);
      load(d, j + d + D);
      list(d, min(j + d + 2 * D, cnt - 1));
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // at most 2 D - 1 units are left, the first D of them loaded
#pragma unroll
  for (int d = 0; d < D; ++d) {
    if (j + d < cnt) mma(d);
    __builtin_amdgcn_sched_barrier(0);
    if (j + d + D < cnt) load(d, j + d + D);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int d = 0; d < D; ++d)
    if (j + d + D < cnt) mma(d);
}

// Row of a 16-row block held in accumulator register r of lane group g: the
// FP64 instruction's order (g + 4 r) or the FP32 one's (4 g + r).
template <typename VT, bool WIDE>
__device__ __forceinline__ int acc_row(int g, int r) {
  return std::is_same<VT, float>::value && !WIDE ? 4 * g + r : g + 4 * r;
}

// Workgroup b runs on XCD b % 8 (round-robin dispatch; each XCD has its own
// L2).  Workgroup b takes item xcd_item(b, n) so that every XCD works through
// one contiguous eighth of the items: neighbouring row blocks, which multiply
// mostly the same vector slices, then share one L2.
__device__ __forceinline__ int xcd_item(int b, int n) {
  constexpr int kXcd = 8;
  const int x = b % kXcd, i = b / kXcd, q = n / kXcd, r = n % kXcd;
  return x * q + min(x, r) + i;
}

// Wave index as a uniform (scalar) value.
__device__ __forceinline__ int wave_uniform() {
  return __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
}

// Waves per workgroup of the interior solves: a row block's tiles are dealt to
// them in turn and their partial products summed in wave order through LDS.
constexpr int kTW = 4;

// One workgroup (TW waves) per block of 16 rows of a tiled matrix:
//   out = base + sum over waves w of (c1 * (units [ptr, split) of wave w applied to x1)
//                                     + c2 * (units [split, ptr+1) of wave w applied to x2))
// (split == nullptr: one part, units [ptr, ptr+1) applied to x1; base may be
// nullptr; a part whose coefficient is 0 is skipped).  All vectors DD layout
// with leading dimension ld, out nrows rows.  Wave w takes units b + w, b + w +
// TW, ...; the wave sums are added in wave order.  With DOT the workgroup also
// writes x1^T out over its rows per column to red.part2 (the step length of the
// CG iteration, from p^T S p); grouped: the last of every kPGroup consecutive
// workgroups also writes the group sum to red.part3, for the update kernel,
// which otherwise reads the block sums themselves.
// Bound (interface rows, 2 320 blocks of 45 units, 32 columns, h = 1/160):
// without the unit and vector loads, matrix instructions and the fixed work of a
// block (column lists, wave sums, dot product) take 50 of the 66 us in FP64,
// 14 us of it fixed; the units are 215 MB.  32-row blocks of aligned 8-column
// units took 78.6 us (FP64) and 56 us (FP32, now 45).  Waves per block (2, 4, 8)
// and units in flight (1 to 4) change it by less than 5 % around 4 and 2.
// run (may be nullptr): the CG loop's flag of columns still
// iterating; when it reads 0 the launch does nothing (the loop's host runs a
// few iterations ahead of the device).  x1f, x2f (FP32 units only; may be
// nullptr): FP32 copies of x1, x2 whose rows the products load instead.
template <typename VT, int NCB, bool DOT, int D, int TW, bool WIDE>
__device__ __forceinline__ void
tile_rows_body(int rb, int nrows, int b, int s, int e, bool split, const int4 *__restrict__ tcol,
               const VT *__restrict__ tval, const double *__restrict__ x1, const double *__restrict__ x2, int ld,
               const double *__restrict__ base, double c1, double c2, double *__restrict__ out, RedBuf red, int nrb,
               const float *__restrict__ x1f, const float *__restrict__ x2f, bool grouped) {
  constexpr int NT = TW * kWave;
  const int wv = wave_uniform(), lane = lane_id(), g = lane >> 4, l16 = lane & 15;
  // one accumulator: with both parts, the second part's products enter the
  // same sums with x2 negated when c2 = -c1 (exact), and the total is scaled by
  // c1; a lone part is scaled by its own coefficient.  Only c2 = +-c1 is
  // served with both parts.
  dbl4 acc[NCB];
#pragma unroll
  for (int q = 0; q < NCB; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[q][r] = 0.0;
  const double sg2 = (c1 != 0.0 && c2 == -c1) ? -1.0 : 1.0;
  const int nel = kT * ld;
  constexpr int NF = (kT * kT * NCB + NT - 1) / NT;   // (ld <= 16 NCB)
  // this thread's output elements; with DOT, their x1 values are loaded now, so
  // that the loads are done when the block's sums are (the dot product then
  // costs no memory round trip after the product)
  double xd[NF];
#pragma unroll
  for (int u = 0; u < NF; ++u) {
    const int el = threadIdx.x + u * NT;
    const int lr = el / ld, row = rb * kT + lr;
    xd[u] = (DOT && el < nel && row < nrows) ? x1[(size_t)row * ld + (el - lr * ld)] : 0.0;
  }
  // the units are dealt to the waves in turn through both parts, from another
  // wave in each row block (a wave keeps its SIMD, so the odd units spread)
  const int w1 = (wv + rb) & (TW - 1), w2 = (w1 - (s - b)) & (TW - 1);
  auto part1 = [&](auto x) { tile_row_acc<NCB, D, WIDE>(b + w1, s, TW, tcol, tval, x, ld, 1.0, acc); };
  auto part2 = [&](auto x) { tile_row_acc<NCB, D, WIDE>(s + w2, e, TW, tcol, tval, x, ld, sg2, acc); };
  if constexpr (std::is_same<VT, float>::value) {
    if (c1 != 0.0) x1f ? part1(x1f) : part1(x1);
    if (split && c2 != 0.0) x2f ? part2(x2f) : part2(x2);
  } else {
    if (c1 != 0.0) part1(x1);
    if (split && c2 != 0.0) part2(x2);
  }
  const double cf = c1 != 0.0 ? c1 : c2;
  __shared__ double part[TW * kT * kT * NCB];    // ld <= 16 NCB
#pragma unroll
  for (int q = 0; q < NCB; ++q) {
    const int col = NCB * l16 + q;
#pragma unroll
    for (int r = 0; r < 4; ++r)                  // row of the block held in register r
      if (col < ld) part[(wv * kT + acc_row<VT, WIDE>(g, r)) * ld + col] = cf * acc[q][r];
  }
  __syncthreads();
  double fin[NF], vo[NF];
#pragma unroll
  for (int u = 0; u < NF; ++u) {
    const int el = threadIdx.x + u * NT;
    fin[u] = vo[u] = 0.0;
    if (el < nel) {
      const int lr = el / ld, col = el - lr * ld, row = rb * kT + lr;
      double v = part[el];
#pragma unroll
      for (int w = 1; w < TW; ++w) v += part[w * nel + el];
      if (row < nrows) {
        const size_t o = (size_t)row * ld + col;
        v += base ? base[o] : 0.0;
        vo[u] = v;
        if (DOT) fin[u] = v * xd[u];
        else out[o] = v;
      }
    }
  }
  if (!DOT) return;
  // (the output is stored after this workgroup has counted itself done: the
  // completion wait before the count then covers the partial only)
  auto store_out = [&]() {
#pragma unroll
    for (int u = 0; u < NF; ++u) {
      const int el = threadIdx.x + u * NT;
      const int lr = el / ld, row = rb * kT + lr;
      if (el < nel && row < nrows) out[(size_t)row * ld + (el - lr * ld)] = vo[u];
    }
  };
  // x1^T out over the block's 16 rows, rows 8 apart added first, then 4, 2, 1: a
  // thread's elements lie in one column, NT / ld rows apart (those further apart
  // than that are added in registers), the rest goes through LDS
  __shared__ double dsum[NT];
  const int per = max(1, nel / NT);              // elements of a thread
#pragma unroll
  for (int h = NF / 2; h >= 1; h /= 2)
    if (h < per)
#pragma unroll
      for (int u = 0; u < h; ++u) fin[u] += fin[u + h];
  dsum[threadIdx.x] = fin[0];
  __syncthreads();
  double sm = 0.0;
  if ((int)threadIdx.x < ld) {
    const int R = kT / per;
    double u[kT];
#pragma unroll
    for (int r = 0; r < kT; ++r) u[r] = r < R ? dsum[r * ld + threadIdx.x] : 0.0;
#pragma unroll
    for (int h = kT / 2; h >= 1; h /= 2)
      if (h < R)
#pragma unroll
        for (int r = 0; r < h; ++r) u[r] += u[r + h];
    sm = u[0];
  }
  if (!grouped) {
    if ((int)threadIdx.x < ld) red.part2[(size_t)rb * ld + threadIdx.x] = sm;
    store_out();
    return;
  }
  if ((int)threadIdx.x < ld) store_partial(red.part2 + (size_t)rb * ld + threadIdx.x, sm);
  const int grp = rb / kPGroup;
  const int members = min(kPGroup, nrb - grp * kPGroup);
  __shared__ int lflag;
  unsigned *cnt = red.gcount + (size_t)grp * kCounterStride;
  const bool last = last_of(cnt, (unsigned)members, &lflag);
  store_out();
  if (!last) return;
  // (read by the next launch: no completion wait)
  group_sums_store(red.part2, nrb, ld, grp, red.part3, wv, TW, false);
  __syncthreads();
  if (threadIdx.x == 0) reset_counter(cnt);
}

template <typename VT, int NCB, bool DOT, int D, int TW, bool WIDE>
__global__ void __launch_bounds__(TW * kWave, kMfmaWaves)
k_tile_rows(int nrb, int nrows, const int *__restrict__ ptr, const int *__restrict__ split,
            const int4 *__restrict__ tcol, const VT *__restrict__ tval, const double *__restrict__ x1,
            const double *__restrict__ x2, int ld, const double *__restrict__ base,
            double c1, double c2, double *__restrict__ out, RedBuf red, const int *__restrict__ run,
            const float *__restrict__ x1f, const float *__restrict__ x2f, int grouped) {
  const int rb = xcd_item(blockIdx.x, nrb);
  // (loaded beside the flag, not after it: one memory round trip less)
  const int b = ptr[rb], e = ptr[rb + 1], s = split ? split[rb] : e;
  if (run && *run == 0) return;                  // every column of the CG loop has stopped
  tile_rows_body<VT, NCB, DOT, D, TW, WIDE>(rb, nrows, b, s, e, split != nullptr, tcol, tval, x1, x2, ld, base, c1, c2,
                                      out, red, nrb, x1f, x2f, grouped != 0);
}

// ------------------------------------------------- vector step of a tiled CG --
// Between q = S p and the next product the vectors take two passes:
//   k_tile_update     alpha from the npq p^T q sums pqs; r -= alpha q, z = D^-1 r and
//                     the partial sums of r.z and r.r;
//   k_tile_direction  beta from those; x += alpha p, p = z + beta p, the column
//                     state -- and, in the same launch, u = K_IG z, which needs
//                     neither: with w_k = K_II^-1 K_IG z_k + beta w_{k-1} (the
//                     recurrence of p through a linear map; k_dense_tiles adds
//                     the second term) the K_IG product no longer waits for p.
// An iteration is four launches (k_dense_tiles, k_tile_rows on the interface
// rows, these two) instead of five, the row blocks of K_IG run beside the
// direction's reductions, and the vectors are read and written 9 times instead
// of 10.  Bound: HBM and the reductions' load latency.  Peridynamic batch (37 114
// rows x 32 columns): K_IG 21.7 + update 18.9 + direction 12.2 us before, update
// 9.4 + direction with K_IG 28 us now; fractional system (5 181 x 8): 6.6 + 6.8 +
// 5.7 us before, 4.8 + 6.2 us now.
//
// A workgroup of the update takes kSlab rows x cw columns (cw = min(ld, 16): 128-byte
// row segments), so narrow systems still fill the chip; a thread keeps one
// column.  Sums over rows and slabs run in one order for every width.
constexpr int kTileCols = 16;

// out[t][c] of CW columns from the slab's terms in registers: element k of
// thread t is row t / CW + k 256 / CW.  Pairs of rows SR / 2 apart are added
// first, then SR / 4, ...: the levels within a thread, then one thread per
// column and dot from LDS.  lds: 2 kBlock doubles.
template <int SR, int CW>
__device__ __forceinline__ void slab_sums2(double (&a)[SR * CW / kBlock], double (&b)[SR * CW / kBlock], double *lds,
                                           double *outa, double *outb) {
  constexpr int E = SR * CW / kBlock, R = kBlock / CW;
#pragma unroll
  for (int h = E / 2; h >= 1; h /= 2)
#pragma unroll
    for (int k = 0; k < h; ++k) {
      a[k] += a[k + h];
      b[k] += b[k + h];
    }
  lds[threadIdx.x] = a[0];
  lds[kBlock + threadIdx.x] = b[0];
  __syncthreads();
  if (threadIdx.x < 2 * CW) {
    const int t = threadIdx.x / CW, c = threadIdx.x % CW;
    double u[R];
#pragma unroll
    for (int r = 0; r < R; ++r) u[r] = lds[t * kBlock + r * CW + c];
#pragma unroll
    for (int h = R / 2; h >= 1; h /= 2)
#pragma unroll
      for (int r = 0; r < h; ++r) u[r] += u[r + h];
    (t ? outb : outa)[c] = u[0];
  }
}

// Sum over i < n of src[i * ld] for column c of the calling thread's column
// (thread t: column t % cw): sixteen threads take i = 0, 16, .. / 1, 17, .. /
// ... in order, and every thread of the column adds the sixteen in order.
// lds: 16 kTileCols doubles, free on entry and on return of the next barrier.
__device__ __forceinline__ double column_sum(const double *__restrict__ src, int n, int ld, int cw, double *lds) {
  const int c = threadIdx.x & (cw - 1), gi = threadIdx.x / cw;
  if (gi < 16) {
    double s = 0.0;
    constexpr int U = 8;                         // loads in flight
    for (int i0 = gi; i0 < n; i0 += 16 * U) {
      double v[U];
#pragma unroll
      for (int k = 0; k < U; ++k) v[k] = i0 + 16 * k < n ? src[(size_t)(i0 + 16 * k) * ld + c] : 0.0;
#pragma unroll
      for (int k = 0; k < U; ++k) s += v[k];
    }
    lds[gi * cw + c] = s;
  }
  __syncthreads();
  double s = lds[c];
#pragma unroll
  for (int k = 1; k < 16; ++k) s += lds[k * cw + c];
  return s;
}

// mode 1: the step; mode 3: residual replacement (the columns that stepped
// take the residual given in q; x and p are kept).  XUP: also x += alpha p (a
// step that is followed by a replacement, which multiplies the new x).  The
// workgroups of slab 0 record the state the step started from, its step
// lengths and breakdown marks.
template <int SR, int CW, bool XUP>
__global__ void __launch_bounds__(kBlock)
k_tile_update(int mode, int nrows, int ld, const double *__restrict__ dinv, double *__restrict__ x,
              double *__restrict__ r, double *__restrict__ z, const double *__restrict__ p,
              const double *__restrict__ q, RedBuf red, ColState st, const double *__restrict__ pqs, int npq,
              float *__restrict__ z32, const int *__restrict__ run) {
  constexpr int E = SR * CW / kBlock, R = kBlock / CW;
  __shared__ double lds[2 * kBlock];
  const int ncb = ld / CW, cb = blockIdx.x % ncb, slab = blockIdx.x / ncb;
  const int c0 = cb * CW, col = c0 + threadIdx.x % CW;
  const int row0 = slab * SR + threadIdx.x / CW;
  double rv[E], qv[E], dv[E], xv[E], pv[E];
  // (the flag is looked at once the loads are under way)
  const int go = run ? *run : 1;
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const int j = row0 + k * R;
    rv[k] = qv[k] = xv[k] = pv[k] = 0.0;
    dv[k] = 1.0;
    if (j < nrows) {
      const size_t o = (size_t)j * ld + col;
      rv[k] = r[o];
      qv[k] = q[o];
      if (XUP && mode == 1) {
        xv[k] = x[o];
        pv[k] = p[o];
      }
      if (dinv) dv[k] = dinv[j];
    }
  }
  if (go == 0) {                                 // every column has stopped, or none is due (mode 3)
    if (mode == 1 && slab == 0 && threadIdx.x < CW) st.act_prev[col] = 0;     // no column takes this step
    return;
  }
  int act;
  double al = 0.0;
  if (mode == 1) {
    const double pq = column_sum(pqs + c0, npq, ld, CW, lds);
    const int act0 = st.active[col];
    const double rz0 = st.rz[col];
    act = act0 && pq > 0.0;
    if (act) al = rz0 / pq;
    if (slab == 0 && threadIdx.x < CW) {
      st.rz_prev[col] = rz0;
      st.act_prev[col] = act0;
      st.brk[col] = act0 && !act;
      st.alpha[col] = al;
    }
    __syncthreads();                             // the sums are read: lds is reused below
  } else {
    act = st.act_prev[col] && !st.brk[col];
    if (blockIdx.x == 0 && threadIdx.x == 0) st.flag[3] = 1;     // read by the direction launch
  }
  double rz[E], rr[E];
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const int j = row0 + k * R;
    rz[k] = rr[k] = 0.0;
    if (j < nrows) {
      const size_t o = (size_t)j * ld + col;
      double rn = rv[k];
      if (act) {
        rn = mode == 1 ? fma(-al, qv[k], rn) : qv[k];
        r[o] = rn;
        if (XUP && mode == 1) x[o] = fma(al, pv[k], xv[k]);
      }
      const double zn = dinv ? dv[k] * rn : rn;
      if (act) {
        z[o] = zn;
        if (z32) z32[o] = (float)zn;
      }
      rz[k] = rn * zn;
      rr[k] = rn * rn;
    }
  }
  slab_sums2<SR, CW>(rz, rr, lds, red.part0 + (size_t)slab * ld + c0, red.part1 + (size_t)slab * ld + c0);
}

// Nothing happens unless some column took the step (act_prev, written by the
// update; the loop flag itself is rewritten by this launch).  Workgroup 0: the
// column state of the step from the nsl slab sums (and the state it started
// from), published to host_nact (active columns + 1); no other workgroup of the
// launch reads what it writes.  Workgroups 1 .. nrb: u = K_IG z, one row block each
// (four waves).  The others: x += alpha p (unless the update did: xup = 0) and
// p = z + beta p over kDirSlab rows x cw columns.  (The row blocks take longest
// and come first: the short direction workgroups then fill the places beside
// them.)
constexpr int kDirSlab = 64;
template <typename VT, int NCB>
__global__ void __launch_bounds__(kBlock, kMfmaWaves)
k_tile_direction(int nrows, int ld, const double *__restrict__ z, double *__restrict__ p,
                 double *__restrict__ x, int xup, RedBuf red, ColState st, int nsl, int *__restrict__ host_nact,
                 float *__restrict__ p32, double drop2, int nrb, int nI,
                 const int *__restrict__ ptr, const int4 *__restrict__ tcol, const VT *__restrict__ tval,
                 double *__restrict__ u, const float *__restrict__ z32) {
  const bool none = __ballot(lane_id() < ld && st.act_prev[lane_id()] != 0) == 0;    // no column stepped
  if (blockIdx.x > 0 && (int)blockIdx.x <= nrb) {
    const int rb = xcd_item((int)blockIdx.x - 1, nrb);
    const int b = ptr[rb], e = ptr[rb + 1];
    if (none) return;
    tile_rows_body<VT, NCB, false, 2, 4, false>(rb, nI, b, e, e, false, tcol, tval, z, nullptr, ld, nullptr, 1.0, 0.0, u,
                                         red, nrb, z32, nullptr, false);
    return;
  }
  __shared__ double lds[16 * kTileCols];
  const int cw = min(ld, kTileCols), ncb = ld / cw;
  if (blockIdx.x > 0) {
    constexpr int E = kDirSlab * kTileCols / kBlock;
    const int d = (int)blockIdx.x - 1 - nrb, cb = d % ncb, slab = d / ncb;
    const int col = cb * cw + (threadIdx.x & (cw - 1)), R = kBlock / cw;
    const int row0 = slab * kDirSlab + threadIdx.x / cw, row1 = min(nrows, (slab + 1) * kDirSlab);
    const int act0 = st.act_prev[col], brk = st.brk[col];
    const double rzp = st.rz_prev[col], al = st.alpha[col];
    double zv[E], pv[E], xv[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int j = row0 + k * R;
      zv[k] = pv[k] = xv[k] = 0.0;
      if (j < row1) {
        const size_t o = (size_t)j * ld + col;
        zv[k] = z[o];
        pv[k] = p[o];
        if (xup) xv[k] = x[o];
      }
    }
    if (none) return;
    const double rz = column_sum(red.part0 + cb * cw, nsl, ld, cw, lds);
    if (!act0 || brk) return;
    const double beta = rz / rzp;
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const int j = row0 + k * R;
      if (j < row1) {
        const size_t o = (size_t)j * ld + col;
        const double pn = fma(beta, pv[k], zv[k]);
        p[o] = pn;
        if (p32) p32[o] = (float)pn;
        if (xup) x[o] = fma(al, pv[k], xv[k]);
      }
    }
    return;
  }
  // workgroup 0: the column state
  if (none) {                                    // every column had stopped: nothing changes, report none active
    if (threadIdx.x == 0 && host_nact) __hip_atomic_store(host_nact, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    return;
  }
  __shared__ int sact[kMaxLd], sdue[kMaxLd];
  for (int cb = 0; cb < ncb; ++cb) {
    const double rz = column_sum(red.part0 + cb * cw, nsl, ld, cw, lds);
    __syncthreads();
    const double rr = column_sum(red.part1 + cb * cw, nsl, ld, cw, lds);
    __syncthreads();
    if ((int)threadIdx.x < cw) {
      const int c = cb * cw + threadIdx.x;
      const int act0 = st.act_prev[c], brk = st.brk[c];
      int act = 0;
      double beta = 0.0;
      if (act0 && brk) st.flag[0] = 1;           // breakdown: p^T q <= 0
      // residual replacement: the reference norm after one, and whether the
      // column is due for the next.  A replaced residual no smaller than the
      // one replaced before means the directions make no progress on the
      // true residual (operators too inaccurate for the system): the column
      // stops, and the FP64 check of its residual decides what follows.
      double ref = st.ref2[c];
      if (act0 && !brk) {
        beta = rz / st.rz_prev[c];
        act = rr > st.stop2[c] ? 1 : 0;
        st.iters[c] += 1;
        st.rz[c] = rz;
        if (st.flag[3]) {                        // replaced in this step
          if (!(rr < ref)) act = 0;
          ref = rr;
          st.ref2[c] = ref;
        }
      }
      st.beta[c] = beta;
      sdue[c] = (act && rr < drop2 * ref) ? 1 : 0;
      sact[c] = act;
      st.active[c] = act;
      st.nrm2[c] = rr;
    }
  }
  __syncthreads();
  if (threadIdx.x < kWave) {
    const int lane = threadIdx.x;
    int na = lane < ld ? sact[lane] : 0;
    int nd = lane < ld ? sdue[lane] : 0;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
      na += __shfl_xor(na, o, kWave);
      nd += __shfl_xor(nd, o, kWave);
    }
    if (lane == 0) {
      if (st.flag[0]) na = 0;                    // breakdown ends the loop
      st.flag[1] = na > 0 ? 1 : 0;
      st.flag[2] = (na > 0 && nd > 0) ? 1 : 0;
      st.flag[3] = 0;
      if (host_nact) __hip_atomic_store(host_nact, na + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
}

// Interior solve w = base + sign * K_II^-1 y on the matrix cores (or, with the
// blocks K_II themselves, the interior part of a residual): one workgroup per
// work item (subdomain k, 16-row tile I of its block; items[b] is the item of
// workgroup b, arranged by the host so that all items of a subdomain run on one
// XCD, and k = -1 pads).  The blocks are packed
// by k_pack_tiles into 16x16 tiles in the A-operand order, block row I of
// subdomain k at toff[k] + I * nt_k * 256 (nt_k = ceil(n_k / 16) tiles per
// row, zero padded).  Wave w applies the tiles J = w, w + kTW, ... to the
// 16-row slices of y; the wave sums are added in wave order.  FP64 blocks:
// v_mfma_f64_16x16x4f64; FP32 blocks (mixed path): v_mfma_f32_16x16x4f32 with
// FP32 operands and accumulation, the wave sums added in FP64; WIDE: FP32 blocks
// widened, on the FP64 instruction with FP64 y and sums.  beta (may be
// nullptr): w += beta w_before per column (the CG's recurrence, k_tile_direction).
template <typename MT> struct DenseAcc;
template <> struct DenseAcc<double> {
  typedef dbl4 acc_t;
  static __device__ __forceinline__ int row(int g, int r) { return g + 4 * r; }
};
template <> struct DenseAcc<float> {
  typedef flt4 acc_t;
  static __device__ __forceinline__ int row(int g, int r) { return 4 * g + r; }
};

// A operand of a packed interior-block tile (layout of TileLayout<MT>).
template <typename MT> struct TileAT;
template <> struct TileAT<double> {
  typedef double v2 __attribute__((ext_vector_type(2)));
  static __device__ __forceinline__ void load(const double *tile, int lane, double (&a)[4]) {
    const v2 u = *(const v2 *)(tile + 2 * lane);
    const v2 v = *(const v2 *)(tile + 128 + 2 * lane);
    a[0] = u[0]; a[1] = u[1]; a[2] = v[0]; a[3] = v[1];
  }
};
template <> struct TileAT<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ void load(const float *tile, int lane, float (&a)[4]) {
    const v4 v = *(const v4 *)(tile + 4 * lane);
    a[0] = v[0]; a[1] = v[1]; a[2] = v[2]; a[3] = v[3];
  }
};

template <typename MT, int NCB, bool WIDE = false>
__global__ void __launch_bounds__(kTW * kWave, kMfmaWaves)
k_dense_tiles(int nall, const int2 *__restrict__ items, const MT *__restrict__ packed,
              const long long *__restrict__ toff, const int *__restrict__ ioff,
              const int *__restrict__ ni, const double *__restrict__ y, int ld,
              const double *__restrict__ base, double sign, double *__restrict__ w,
              const int *__restrict__ run, float *__restrict__ w32, const double *__restrict__ beta) {
  const int wv = wave_uniform(), lane = lane_id(), g = lane >> 4, l16 = lane & 15;
  const int2 item = items[blockIdx.x];
  if (run && *run == 0) return;                  // every column of the CG loop has stopped
  if (item.x < 0) return;                        // padding of a short XCD list
  const int k = item.x, r0 = item.y * kT;
  const int n = ni[k], i0 = ioff[k];
  // this thread's previous w and beta, loaded early
  constexpr int NF = kT * kT * NCB / (kTW * kWave);      // (ld <= 16 NCB)
  double wp[NF], bt[NF];
#pragma unroll
  for (int u = 0; u < NF; ++u) {
    const int el = threadIdx.x + u * kTW * kWave, lr = el / ld, row = r0 + lr;
    wp[u] = bt[u] = 0.0;
    if (beta && el < kT * ld && row < n) {
      bt[u] = beta[el - lr * ld];
      wp[u] = w[(size_t)(i0 + row) * ld + (el - lr * ld)];
    }
  }
  const int nt = (n + kT - 1) / kT;
  const MT *A = packed + toff[k] + (size_t)item.y * nt * 256;
  // y rows past the block (the next subdomain's, or the last row repeated at
  // the end of y) meet the zero padding of the packed tiles
  const double *yb = y + slice_col0<NCB>(l16, ld);
  typedef typename std::conditional<WIDE, double, MT>::type AT;
  typedef typename DenseAcc<AT>::acc_t acc_t;
  acc_t acc[NCB];
#pragma unroll
  for (int q = 0; q < NCB; ++q)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[q][r] = (AT)0;
  auto load = [&](int J, MT (&a)[4], AT (&b)[4][NCB]) {
    TileAT<MT>::load(A + (size_t)J * 256, lane, a);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      double v[NCB];
      slice_row<NCB>(yb + (size_t)min(i0 + J * kT + 4 * s + g, nall - 1) * ld, v);
#pragma unroll
      for (int q = 0; q < NCB; ++q) b[s][q] = (AT)v[q];
    }
  };
  auto mma = [&](const MT (&a)[4], const AT (&b)[4][NCB]) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int q = 0; q < NCB; ++q) acc[q] = mfma16x16x4((AT)a[s], b[s][q], acc[q]);
  };
  // tiles J = wv, wv + kTW, ...: two register buffers in flight, each group of
  // loads kept in program order (see tile_row_acc)
  const int cnt = wv < nt ? (nt - wv + kTW - 1) / kTW : 0;
  if (cnt > 0) {
    MT a0[4], a1[4];
    AT b0[4][NCB], b1[4][NCB];
    load(wv, a0, b0);
    __builtin_amdgcn_sched_barrier(0);
    load(wv + kTW * min(1, cnt - 1), a1, b1);
    __builtin_amdgcn_sched_barrier(0);
    for (int j = 0; j < cnt; j += 2) {
      mma(a0, b0);
      __builtin_amdgcn_sched_barrier(0);
      load(wv + kTW * min(j + 2, cnt - 1), a0, b0);
      __builtin_amdgcn_sched_barrier(0);
      if (j + 1 < cnt) mma(a1, b1);
      __builtin_amdgcn_sched_barrier(0);
      load(wv + kTW * min(j + 3, cnt - 1), a1, b1);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  __shared__ double part[kTW * kT * kT * NCB];   // ld <= 16 NCB
#pragma unroll
  for (int q = 0; q < NCB; ++q) {
    const int c = NCB * l16 + q;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (c < ld) part[(wv * kT + DenseAcc<AT>::row(g, r)) * ld + c] = (double)acc[q][r];
  }
  __syncthreads();
  const int nel = kT * ld;
#pragma unroll
  for (int f = 0; f < NF; ++f) {
    const int el = threadIdx.x + f * kTW * kWave;
    const int lr = el / ld, c = el - lr * ld, row = r0 + lr;
    if (el < nel && row < n) {
      double v = part[el];
#pragma unroll
      for (int u = 1; u < kTW; ++u) v += part[u * nel + el];
      const size_t o = (size_t)(i0 + row) * ld + c;
      double wn = (base ? base[o] : 0.0) + sign * v;
      if (bt[f] != 0.0) wn = fma(bt[f], wp[f], wn);      // (beta = 0: w holds nothing yet)
      w[o] = wn;
      if (w32) w32[o] = (float)wn;           // FP32 copy for the FP32 unit products
    }
  }
}

// Packs column-major dense blocks (n_k x n_k at koff[k]) into the tile order
// of k_dense_tiles: tile (I, J) of block k at toff[k] + (I * nt + J) * 256,
// lane l holding B[16 I + l % 16][16 J + 4 s + l / 16] at position
// TileLayout<T>::pos(l, s).
template <typename T>
__global__ void k_pack_tiles(int nsub, const T *__restrict__ blocks, const long long *__restrict__ koff,
                             const long long *__restrict__ toff, const int *__restrict__ ni,
                             T *__restrict__ packed) {
  const int k = blockIdx.y;
  if (k >= nsub) return;
  const int n = ni[k], nt = (n + kT - 1) / kT;
  const long long tot = (long long)nt * nt * 256;
  const T *B = blocks + koff[k];
  T *P = packed + toff[k];
  for (long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x; e < tot;
       e += (long long)gridDim.x * blockDim.x) {
    const int t = (int)(e / 256), pos = (int)(e % 256);
    const int I = t / nt, J = t % nt, l = TileLayout<T>::lane(pos), s = TileLayout<T>::step(pos);
    const int i = I * kT + (l & 15), j = J * kT + 4 * s + (l >> 4);
    P[e] = (i < n && j < n) ? B[(size_t)j * n + i] : (T)0;
  }
}

}  // namespace dd
