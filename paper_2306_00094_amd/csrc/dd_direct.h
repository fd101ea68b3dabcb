// Interface CG of small interfaces in one launch (gfx950).
//
// With a few hundred interface rows an iteration moves next to nothing: its
// three launches take 16 us on the 1D system (159 interface rows), all of it
// launch and load latency.  The Schur complement itself is then small enough to
// keep: S = K_GG - sum_k K_GI^k (K_II^k)^-1 K_IG^k (eq. subSchurComplement,
// summed as in eq. SchurComplement) is formed once per factorisation as a dense
// matrix, and one workgroup per right-hand side runs the whole preconditioned
// CG on it, with S in registers (up to 192 rows; beyond that the rest is read
// from the L2).  A column never sees the others, so its result does not depend
// on the batch.
#pragma once

#include "dd_kernels.h"

namespace dd {

constexpr int kSchurBlock = 1024;
constexpr int kDirectBlock = 512, kDirectWaves = kDirectBlock / kWave;
// Interfaces served: 384 rows.  S then streams 1.2 MB an iteration from the L2
// through one compute unit: a 1D solve with 370 rows takes 472 us, 526 us in three
// launches an iteration; with 500 rows 822 and 584 us.
constexpr int kDirectRows = 6, kDirectMax = kDirectRows * kWave;
constexpr int kDirectMaxNI = 7680;       // interior rows (one vector in 60 KB of LDS)

inline int direct_ld(int n) { return (n + kWave - 1) / kWave * kWave; }

// Row j of the dense S (N values, zeros up to Np), one workgroup per row: t =
// K_II^-1 K_IG e_j in LDS, then S[j][l] = (K_GG)_lj - (K_GI)_l t, a wave per l.
template <typename VT, typename MT>
__global__ void __launch_bounds__(kSchurBlock)
k_direct_schur(int N, int Np, int NI, const int *__restrict__ ptr, const int *__restrict__ split,
               const int *__restrict__ col, const VT *__restrict__ val, const MT *__restrict__ kinv,
               const long long *__restrict__ koff, const int *__restrict__ ioff, const int *__restrict__ ni,
               const int *__restrict__ rowsub, double *__restrict__ S) {
  extern __shared__ double t[];
  const int j = blockIdx.x;
  for (int i = threadIdx.x; i < NI; i += kSchurBlock) t[i] = 0.0;
  __syncthreads();
  for (int a = split[j]; a < ptr[j + 1]; ++a) {        // (a thread keeps its rows of every subdomain)
    const int r = col[a], k = rowsub[r], i0 = ioff[k], n = ni[k];
    const double v = (double)val[a];
    const MT *m = kinv + koff[k] + (size_t)(r - i0) * n;
    for (int i = threadIdx.x; i < n; i += kSchurBlock) t[i0 + i] = fma(v, (double)m[i], t[i0 + i]);
  }
  __syncthreads();
  const int lane = lane_id();
  for (int l = wave_id(); l < Np; l += kSchurBlock / kWave) {
    double s = 0.0;
    if (l < N) {
      const int mid = split[l];
      for (int a = ptr[l] + lane; a < ptr[l + 1]; a += kWave) {
        const int cc = col[a];
        if (a < mid) s += cc == j ? (double)val[a] : 0.0;
        else s = fma(-(double)val[a], t[cc], s);
      }
      s = wave_sum(s);
    }
    if (lane == 0) S[(size_t)j * Np + l] = s;
  }
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
