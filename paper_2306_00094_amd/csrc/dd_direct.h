// Interface CG of small interfaces in one launch (gfx950).
//
// With a few hundred interface rows an iteration moves next to nothing: its
// three launches take 16 us on the 1D system (159 interface rows), all of it
// launch and load latency.  The Schur complement itself is then small enough to
// keep: S = K_GG - sum_k K_GI^k (K_II^k)^-1 K_IG^k (eq. subSchurComplement,
// summed as in eq. SchurComplement) is formed once per factorisation, by the first
// solve after it, as a dense matrix, and one workgroup per right-hand side runs the
// whole preconditioned
// CG on it, with S in registers (up to 192 rows; beyond that the rest is read
// from the L2).  A column never sees the others, so its result does not depend
// on the batch.
#pragma once

#include "dd_kernels.h"

namespace dd {

constexpr int kDirectBlock = 512, kDirectWaves = kDirectBlock / kWave;
// Interfaces served: 384 rows.  S then streams 1.2 MB an iteration from the L2
// through one compute unit: a 1D solve with 370 rows takes 472 us, 526 us in three
// launches an iteration; with 500 rows 822 and 584 us.
// The first solve after a factorisation also forms S.  FP64, us, one column (first
// solve / later ones / three launches an iteration): 1D with 159 rows 115 / 95 / 486,
// 315 rows 406 / 364 / 517, 371 rows on 8 strips 616 / 602 / 595 (8 columns 657 / 630
// / 1250).  It pays from the first solve on, but for matrices with hundreds of
// entries a row and few iterations: 384 rows of 1 100 entries 336 / 184 / 250, paid
// back by the third solve; 7 interiors of 960 rows coupled to 40 % of them (6 720
// rows, the largest measured: hence the limit) 651 / 195 / 354, by the third too.
constexpr int kDirectRows = 6, kDirectMax = kDirectRows * kWave;
constexpr int kDirectMaxNI = 7680;       // interior rows

inline int direct_ld(int n) { return (n + kWave - 1) / kWave * kWave; }

// S is formed in two launches.  k_direct_columns: T_k = (K_II^k)^-1 K_IG^k on the
// matrix cores, one wave per 16 rows and kStrips strips of 16 interface columns of
// the packed K_IG^k (the items of k_schur_wsq, whose row tiles without entries are
// skipped); K_II^-1 symmetric, its rows are read as columns.  FP32 operators are
// widened, their K_IG rounded as the CG's is.  T (NI x Np) is stored by interior
// rows and interface columns gcol of the strips' columns; it is zero elsewhere.
// Bound: the latency of a wave's row of tiles (six dependent loads, then four tiles a
// step).  1D, 159 rows (4 blocks of 216): 12 us; 315 rows (4 of 433): 24 us.
template <typename T>
__global__ void __launch_bounds__(kBlock, kMfmaWaves)
k_direct_columns(const T *__restrict__ kinv, const double *__restrict__ packed, const long long *__restrict__ koff,
                 const long long *__restrict__ voff, const int *__restrict__ ni, const int *__restrict__ goff,
                 const int *__restrict__ ioff, const int4 *__restrict__ items, const int *__restrict__ gcol, int Np,
                 double *__restrict__ T_) {
  typedef typename Vec4<T>::type V4;
  typedef V4 V4u __attribute__((aligned(sizeof(T))));
  const int4 it = items[blockIdx.x];
  if (it.x < 0) return;                      // padding of the item list
  const int k = it.x, J = it.y, kl = it.w;
  const int n = ni[k], nt = (n + 15) / 16, g0 = goff[k], ng = goff[k + 1] - g0, ns = (ng + 15) / 16;
  const int lane = lane_id(), c = lane % 16, g = lane / 16, I = blockIdx.y * kWavesPerBlock + wave_id();
  if (I >= nt) return;
  const T *xr = kinv + koff[k] + (size_t)min(16 * I + c, n - 1) * n;   // (rows past the end are not stored)
  const double *V[kStrips];
  dbl4 acc[kStrips];
#pragma unroll
  for (int s = 0; s < kStrips; ++s) {        // (past the last strip: that strip again, not stored)
    V[s] = packed + voff[k] + (size_t)min(J + s, ns - 1) * nt * 256 + 4 * lane;
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[s][r] = 0.0;
  }
  auto mma = [&](int K, const V4 &a) {
#pragma unroll
    for (int s = 0; s < kStrips; ++s) {
      const dbl4 b = *reinterpret_cast<const dbl4 *>(V[s] + (size_t)K * 256);
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[s] = mfma16x16x4((double)a[t], (double)(T)b[t], acc[s]);
    }
  };
  int K = it.z;
  const int kw = min(kl + 1, n / 16);        // whole tiles of 16 columns
  for (; K + 3 < kw; K += 4) {               // four tiles per step: their loads go out together
    V4 a[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u] = *reinterpret_cast<const V4u *>(xr + 16 * (K + u) + 4 * g);
#pragma unroll
    for (int u = 0; u < 4; ++u) mma(K + u, a[u]);
  }
  for (; K <= kl; ++K) {
    const int q = 16 * K + 4 * g;
    V4 a;
#pragma unroll
    for (int t = 0; t < 4; ++t) a[t] = q + t < n ? xr[q + t] : T(0);
    mma(K, a);
  }
#pragma unroll
  for (int s = 0; s < kStrips; ++s) {
    const int jl = 16 * (J + s) + c;
    if (jl >= ng) continue;
    double *out = T_ + (size_t)(ioff[k] + 16 * I) * Np + gcol[g0 + jl];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (16 * I + g + 4 * r < n) out[(size_t)(g + 4 * r) * Np] = acc[s][r];
  }
}

// Row l of S, one workgroup per row (those past N: zeros): thread j of a group of Np
// sums (K_GG)_lj - sum_i (K_GI)_li T_ij, the entries staged in LDS and dealt to the
// groups kSchurFly at a time (that many loads in flight), the groups added in order.
// Stored at S[j][l], the operand k_direct_cg multiplies p_j with.
// Bound: load latency (a pass of the entry loop per kSchurFly entries of a group).  1D,
// 159 rows: 7 us, 315 rows: 17 us.  Both launches: 20 and 41 us, against 28 and 90 us
// for one workgroup per row that went through the columns of K_II^-1 one by one, and
// 80 against 570 us with 60 rows of 1 150 entries.
constexpr int kSchurFly = 16, kSchurBlock = 512;
template <typename VT>
__global__ void __launch_bounds__(kSchurBlock)
k_direct_schur(int N, int Np, const int *__restrict__ ptr, const int *__restrict__ split, const int *__restrict__ col,
               const VT *__restrict__ val, const double *__restrict__ T_, double *__restrict__ S) {
  __shared__ double sval[kSchurBlock], part[kSchurBlock];
  __shared__ int scol[kSchurBlock];
  const int l = blockIdx.x, nthr = blockDim.x, t = threadIdx.x, grp = t / Np, j = t - grp * Np, ngrp = nthr / Np;
  double s = 0.0;
  if (l < N) {
    const int b = ptr[l], mid = split[l], e = ptr[l + 1];
    int repeats = 0;                               // (a column given twice, or out of order)
    for (int a = b + 1 + t; a < mid; a += nthr) repeats |= col[a] <= col[a - 1];
    part[t] = 0.0;
    if (!__syncthreads_or(repeats)) {
      for (int a = b + t; a < mid; a += nthr) part[col[a]] = (double)val[a];
      __syncthreads();
      if (grp == 0) s = part[j];
    }
    else
      for (int a0 = b; a0 < mid; a0 += nthr) {
        __syncthreads();
        if (a0 + t < mid) {
          scol[t] = col[a0 + t];
          sval[t] = (double)val[a0 + t];
        }
        __syncthreads();
        for (int a = grp; a < min(nthr, mid - a0); a += ngrp) s += scol[a] == j ? sval[a] : 0.0;
      }
    for (int a0 = mid; a0 < e; a0 += nthr) {
      __syncthreads();                             // the entries before are used
      if (a0 + t < e) {
        scol[t] = col[a0 + t];
        sval[t] = (double)val[a0 + t];
      }
      __syncthreads();
      const int cnt = min(nthr, e - a0);
      for (int a = grp * kSchurFly; a < cnt; a += ngrp * kSchurFly) {
        double m[kSchurFly];
#pragma unroll
        for (int u = 0; u < kSchurFly; ++u) m[u] = a + u < cnt ? T_[(size_t)scol[a + u] * Np + j] : 0.0;
#pragma unroll
        for (int u = 0; u < kSchurFly; ++u)
          if (a + u < cnt) s = fma(-sval[a + u], m[u], s);
      }
    }
    __syncthreads();                               // (part was read as the K_GG row)
    part[t] = s;
    __syncthreads();
    for (int g = 1; grp == 0 && g < ngrp; ++g) s += part[g * Np + j];
  }
  if (grp == 0 && j < N) S[(size_t)j * Np + l] = s;
}

// Sum over the wave in lane 63 (row shifts, then row broadcasts: no LDS
// crossbar, whose round trips would be most of an iteration).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, ROWS, 0xf, false);
  return v + __hiloint2double(hi, lo);
}
__device__ __forceinline__ double wave_sum_63(double v) {
  v = dpp_add<0x111, 0xf>(v);            // row_shr:1
  v = dpp_add<0x112, 0xf>(v);            // row_shr:2
  v = dpp_add<0x114, 0xf>(v);            // row_shr:4
  v = dpp_add<0x118, 0xf>(v);            // row_shr:8
  v = dpp_add<0x142, 0xa>(v);            // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xc>(v);            // row_bcast:31 into rows 2 and 3
  return v;
}

// CG on S x = r0 (x0 = 0, z = D^-1 r) for column blockIdx.x, with the stopping
// rule and the column state of k_cg_update.  Wave w multiplies its share of the
// columns of S, lane l the rows l, l + 64, ... (R of them: one p_j from LDS
// serves R products); up to 192 rows a share stays in registers, above it is
// read again every iteration.  The wave sums are added in wave order by the
// thread that owns the row (thread i < N keeps x, r, z and p of row i).  Bound:
// LDS and barrier latency (four barriers an iteration), above 192 rows the loads
// of S.  1D system, 159 rows: 1.4 us an iteration, against 16 us in three
// launches; 315 rows: 12 us.
template <int R>
__global__ void __launch_bounds__(kDirectBlock, 2)
k_direct_cg(int N, const double *__restrict__ S, int ld, int nrhs, const double *__restrict__ dinv,
            const double *__restrict__ r0, double *__restrict__ x, ColState st, int max_it) {
  constexpr int Np = R * kWave, J = Np / kDirectWaves;      // rows, columns of a share at most
  constexpr bool REG = R <= 3;
  __shared__ double sp[Np + J];
  __shared__ double part[kDirectWaves * Np];
  __shared__ double red[2][2][R];
  const int c = blockIdx.x, i = threadIdx.x, wv = wave_id(), lane = lane_id();
  const int per = (N + kDirectWaves - 1) / kDirectWaves, j0 = min(wv * per, N), j1 = min(N, j0 + per);
  const bool own = i < N;
  double s[REG ? J : 1][R];
  if constexpr (REG) {
#pragma unroll
    for (int u = 0; u < J; ++u)
#pragma unroll
      for (int h = 0; h < R; ++h) s[u][h] = j0 + u < j1 ? S[(size_t)(j0 + u) * Np + h * kWave + lane] : 0.0;
  }
  for (int k = i; k < Np + J; k += kDirectBlock) sp[k] = 0.0;
  double r = own ? r0[(size_t)i * ld + c] : 0.0, xv = 0.0;
  const double d = own && dinv ? dinv[i] : 1.0;
  // sums over the owners (waves 0 .. R - 1), for every thread
  auto sums = [&](int buf, double a, double b, double &ta, double &tb) {
    if (wv < R) {
      a = wave_sum_63(a);
      b = wave_sum_63(b);
      if (lane == kWave - 1) {
        red[buf][0][wv] = a;
        red[buf][1][wv] = b;
      }
    }
    __syncthreads();
    ta = red[buf][0][0];
    tb = red[buf][1][0];
#pragma unroll
    for (int w = 1; w < R; ++w) {
      ta += red[buf][0][w];
      tb += red[buf][1][w];
    }
  };
  double z = d * r, rz, rr, p = z;
  __syncthreads();
  if (own) sp[i] = p;
  sums(0, r * z, r * r, rz, rr);
  const double stop2 = st.stop2[c];
  bool active = c < nrhs && rr > stop2, broke = false;
  int it = 0;
  while (active && it < max_it) {                      // (uniform over the workgroup)
    __syncthreads();
    double acc[R];
#pragma unroll
    for (int h = 0; h < R; ++h) acc[h] = 0.0;
    if constexpr (REG) {
#pragma unroll
      for (int u = 0; u < J; ++u) {                    // (past the share: zeros)
        const double pj = sp[j0 + u];
#pragma unroll
        for (int h = 0; h < R; ++h) acc[h] = fma(s[u][h], pj, acc[h]);
      }
    } else {
      constexpr int U = 8;                             // columns in flight
#pragma unroll 1
      for (int j = j0; j < j1; j += U) {
        double v[U][R];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int h = 0; h < R; ++h) v[u][h] = S[(size_t)min(j + u, N - 1) * Np + h * kWave + lane];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const double pj = j + u < j1 ? sp[j + u] : 0.0;
#pragma unroll
          for (int h = 0; h < R; ++h) acc[h] = fma(v[u][h], pj, acc[h]);
        }
      }
    }
#pragma unroll
    for (int h = 0; h < R; ++h) part[wv * Np + h * kWave + lane] = acc[h];
    __syncthreads();
    double q = 0.0, pq, unused;
    if (own) {
#pragma unroll
      for (int w = 0; w < kDirectWaves; ++w) q += part[w * Np + i];
    }
    sums(1, p * q, 0.0, pq, unused);
    if (!(pq > 0.0)) {                                 // p^T S p <= 0
      broke = true;
      break;
    }
    const double al = rz / pq;
    xv = fma(al, p, xv);
    r = fma(-al, q, r);
    z = d * r;
    double rzn;
    sums(0, r * z, r * r, rzn, rr);
    ++it;
    p = fma(rzn / rz, p, z);
    rz = rzn;
    if (own) sp[i] = p;
    if (rr <= stop2) active = false;
  }
  if (own) x[(size_t)i * ld + c] = xv;
  if (threadIdx.x == 0) {
    st.iters[c] = it;
    st.active[c] = broke ? 0 : (active ? 1 : 0);
    st.nrm2[c] = rr;
    st.rz[c] = rz;
    if (broke) st.flag[0] = 1;
  }
}

}  // namespace dd
