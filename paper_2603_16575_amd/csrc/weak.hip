// Pair screening (eq. s2b) and the weak-pair energies (eqs. osv_weak_k,
// res_weak): what closes the grouped GEMM chains planned by mbe3_screen and
// mbe3_weak_pairs.  Sums run in a fixed order, so every result is reproducible
// bit for bit.
#include "internal.hpp"

namespace mbe3 {

__device__ __forceinline__ double wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// s2b_ij = sum of the squares of the r_i x r_j block S_(i,j) = Q_i^T Q_j at
// k_off, divided by sqrt(r_i r_j).
__global__ __launch_bounds__(256) void s2b_kernel(const WeakPair *__restrict__ wp, int n,
                                                  const double *__restrict__ S,
                                                  double *__restrict__ out) {
  const int lane = threadIdx.x & 63;
  const int p = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (p >= n) return;
  const WeakPair w = wp[p];
  const double *s = S + w.k_off;
  const int m = w.ri * w.rj;
  double acc = 0.0;
  for (int e = lane; e < m; e += 64) acc += s[e] * s[e];
  acc = wave_sum(acc);
  if (lane == 0) out[p] = acc / sqrt((double)w.ri * (double)w.rj);
}

typedef double d4 __attribute__((ext_vector_type(4)));

// e_ij = 4 sum_{a < rank_i, b < rank_j} K~_ab (K~_ab - f_ij D~_ab)
//                                       / (f_ii + f_jj - eps~_i[a] - eps~_j[b])
// with K~ = X_i^T K_(i,j) X_j and D~ = X_i^T (T_ii S_(i,j) + S_(i,j) T_jj) X_j
// = (T_ii^T X_i)^T S X_j + X_i^T S T_jj X_j: the one-block amplitudes in the
// diagonal pairs' bases, contracted with K~.  One workgroup per pair; the
// products from the left are formed here, tile by tile on the matrix cores, so
// that neither they nor a task per pair pass through memory (three lists of
// products and K~, D~ before).  Operands come straight from L2, both with 16
// consecutive doubles per row; bound by that latency.  Measured, 7376 pairs of 30
// x 30: 0.12 ms, with the products it reads 0.27; the seven lists before 0.7.
__global__ __launch_bounds__(256) void weak_energy_kernel(
    const WeakPair *__restrict__ wp, const double *__restrict__ X,
    const double *__restrict__ TX, const double *__restrict__ KX,
    const double *__restrict__ SX, const double *__restrict__ et,
    const int32_t *__restrict__ rank, const double *__restrict__ f, int n_occ,
    double *__restrict__ e) {
  __shared__ double red[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, lq = lane >> 4;
  const WeakPair w = wp[blockIdx.x];
  const int rki = rank[w.i], rkj = rank[w.j];
  const double fii = f[(int64_t)w.i * n_occ + w.i];
  const double fjj = f[(int64_t)w.j * n_occ + w.j];
  const double fij = f[(int64_t)w.i * n_occ + w.j];
  const double *xi = X + w.xi, *ci = TX + w.xi;
  const double *kx = KX + w.t_off, *sx = SX + 2 * w.t_off;
  const double *ei = et + w.ei, *ej = et + w.ej;
  const int ta = w.Di >> 4, tb = w.Dj >> 4;
  double acc = 0.0;
  for (int t = wave; t < ta * tb; t += 4) {
    const int a0 = (t / tb) * 16, b0 = (t % tb) * 16;
    d4 k = {0.0, 0.0, 0.0, 0.0}, d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
    for (int m0 = 0; m0 < w.ri; m0 += 4) {
      const bool in = m0 + lq < w.ri;
      const int64_t m = in ? m0 + lq : 0;  // rows past r_i: zero from both sides
      const double x = xi[m * w.Di + a0 + l16], c = ci[m * w.Di + a0 + l16];
      const double y = kx[m * w.Dj + b0 + l16];
      const double u = sx[m * 2 * w.Dj + b0 + l16], v = sx[m * 2 * w.Dj + w.Dj + b0 + l16];
      const double xa = in ? x : 0.0, ca = in ? c : 0.0;
      const double yb = in ? y : 0.0, ub = in ? u : 0.0, vb = in ? v : 0.0;
      k = __builtin_amdgcn_mfma_f64_16x16x4f64(xa, yb, k, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f64_16x16x4f64(ca, ub, d, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f64_16x16x4f64(xa, vb, d, 0, 0, 0);
    }
    const int b = b0 + l16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int a = a0 + lq + 4 * v;
      if (a < rki && b < rkj)
        acc += k[v] * (k[v] - fij * d[v]) / (fii + fjj - ei[a] - ej[b]);
    }
  }
  acc = wave_sum(acc);
  if (lane == 0) red[wave] = acc;
  __syncthreads();
  if (threadIdx.x == 0) e[blockIdx.x] = 4.0 * ((red[0] + red[1]) + (red[2] + red[3]));
}

// Pairs of one launch: a grid past 2^32 threads wraps without an error.
static constexpr int PAIRS_MAX = 1 << 23;

hipError_t launch_s2b(const WeakPair *wp, int n, const double *S, double *out,
                      hipStream_t s) {
  for (int k = 0; k < n; k += PAIRS_MAX) {
    const int m = n - k < PAIRS_MAX ? n - k : PAIRS_MAX;
    hipLaunchKernelGGL(s2b_kernel, dim3((unsigned)((m + 3) / 4)), dim3(256), 0, s, wp + k, m, S,
                       out + k);
  }
  return hipGetLastError();
}

hipError_t launch_weak_energy(const WeakPair *wp, int n, const double *X, const double *TX,
                              const double *KX, const double *SX, const double *et,
                              const int32_t *rank, const double *f, int n_occ, double *e,
                              hipStream_t s) {
  for (int k = 0; k < n; k += PAIRS_MAX)
    hipLaunchKernelGGL(weak_energy_kernel,
                       dim3((unsigned)(n - k < PAIRS_MAX ? n - k : PAIRS_MAX)), dim3(256), 0, s,
                       wp + k, X, TX, KX, SX, et, rank, f, n_occ, e + k);
  return hipGetLastError();
}

}  // namespace mbe3
