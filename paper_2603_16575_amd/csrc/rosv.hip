// Randomized OSV generation (the paper's randomized OSV section, Alg. 3):
// the pieces between the grouped GEMMs that the C-ABI call plans.
//
//   rosv_tscale_kernel   T_ii[a][b] /= (f_aa + f_bb - 2 f_ii)   (eq. mp2_tkk,
//                        after T = B_D B_D^T over the fitting domain)
//   range_finder_kernel  the adaptive randomized range finder on the rows of
//                        Y = G T: one workgroup per LMO walks the accepted
//                        rows s = 1, 2, ... while the largest of the r
//                        pending row norms exceeds the stopping bound; each
//                        step orthogonalises the first pending row against
//                        the accepted rows (eq. rsvd_za), normalises it,
//                        appends the next sample orthogonalised against the
//                        earlier rows, and removes the new direction from
//                        every pending row
//   rosv_finalize_kernel singular values w = sqrt(eigenvalues of T~ T~^T)
//                        (eq. tii_rsvd via the Gram matrix), rows of
//                        Q_i^T = Q~^T Z (eq. back_q) ordered by decreasing w,
//                        those with w >= l_osv kept
//
// All reductions run in a fixed order (lane-strided partial sums, a xor
// butterfly per wave, the partials in order), so results are
// reproducible bit for bit.
#include "internal.hpp"

namespace mbe3 {

__global__ __launch_bounds__(256) void rosv_tscale_kernel(
    double *__restrict__ T, int i0, int nb, int n_vir, const double *__restrict__ eps,
    const double *__restrict__ f, int n_occ) {
  const int64_t per = (int64_t)n_vir * n_vir;
  const int64_t total = per * nb;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int b = (int)(e / per);
    const int64_t r = e - (int64_t)b * per;
    const int a = (int)(r / n_vir), c = (int)(r - (int64_t)a * n_vir);
    const int i = i0 + b;
    T[e] = T[e] / (eps[a] + eps[c] - 2.0 * f[(int64_t)i * n_occ + i]);
  }
}

hipError_t launch_rosv_tscale(double *T, int i0, int nb, int n_vir, const double *eps,
                              const double *f, int n_occ, hipStream_t s) {
  const int64_t total = (int64_t)nb * n_vir * n_vir;
  if (total <= 0) return hipSuccess;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(rosv_tscale_kernel, dim3((unsigned)blocks), dim3(256), 0, s, T, i0, nb,
                     n_vir, eps, f, n_occ);
  return hipGetLastError();
}

__device__ __forceinline__ double rf_wave_sum(double v) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// <x, y> over n elements by one wave (lane-strided, then the butterfly).
__device__ __forceinline__ double rf_wave_dot(const double *__restrict__ x,
                                              const double *__restrict__ y, int n) {
  double acc = 0.0;
  for (int a = threadIdx.x & 63; a < n; a += 64) acc += x[a] * y[a];
  return rf_wave_sum(acc);
}

// Y: [nb][r + n_max][n_vir] (G T, rows 0..r-1 pending first, then the later
// samples, overwritten as they are orthogonalised; rows s .. s + r - 1 pend at
// step s); Z: [nb][n_max][n_vir] (accepted rows, zero beyond the count);
// rows[b]: accepted count.
//
// Bound by the chain of n_max steps, each a few dependent passes over rows in L2
// with a workgroup per LMO: what counts is the passes and barriers of a step and
// the loads in flight in each.  16 waves; the first pending row and the next
// sample, both taken against the same accepted rows, go through Z together (four
// rows of Z per wave at a time; then half of the threads each); a wave removes the
// new direction from its pending rows and has their next norms without a barrier.
// 96 LMOs, up to 96 rows of 384:
// 4.13 ms with 4 waves and a pass per vector, 1.18 now.
static constexpr int RF_THREADS = 1024;
__global__ __launch_bounds__(RF_THREADS) void range_finder_kernel(
    double *__restrict__ Y, double *__restrict__ Z, int32_t *__restrict__ rows, int r,
    int n_max, int n_vir, double thr) {
  extern __shared__ double rf_sm[];
  double *coef = rf_sm;            // n_max + n_max dot products (first row, next sample)
  double *nrm = coef + 2 * n_max;  // r pending norms
  constexpr int NW = RF_THREADS / 64, HALF = RF_THREADS / 2;
  const int b = blockIdx.x;
  double *Yb = Y + (int64_t)b * (r + n_max) * n_vir;
  double *Zb = Z + (int64_t)b * n_max * n_vir;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int half = threadIdx.x >= HALF, ht = threadIdx.x - half * HALF;
  for (int j = wv; j < r; j += NW) {
    const double *y = Yb + (int64_t)j * n_vir;
    const double q = rf_wave_dot(y, y, n_vir);
    if (lane == 0) nrm[j] = sqrt(q);
  }
  __syncthreads();
  int s = 0;
  for (;;) {
    // largest pending row norm against the stopping bound
    double mx = 0.0;
    for (int j = 0; j < r; ++j) mx = fmax(mx, nrm[j]);
    if (s >= n_max || !(mx > thr)) break;
    double *y = Yb + (int64_t)s * n_vir;
    double *yn = Yb + (int64_t)(r + s) * n_vir;
    double *z = Zb + (int64_t)s * n_vir;
    // y Z^T and yn Z^T over the s accepted rows
    for (int k0 = 4 * wv; k0 < s; k0 += 4 * NW) {
      const double *zk[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) zk[u] = Zb + (int64_t)(k0 + u < s ? k0 + u : s - 1) * n_vir;
      double cy[4] = {0.0, 0.0, 0.0, 0.0}, cn[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
      for (int a = lane; a < n_vir; a += 64) {
        const double ya = y[a], na = yn[a];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const double za = zk[u][a];
          cy[u] += ya * za;
          cn[u] += na * za;
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        cy[u] = rf_wave_sum(cy[u]);
        cn[u] = rf_wave_sum(cn[u]);
        if (lane == 0 && k0 + u < s) {
          coef[k0 + u] = cy[u];
          coef[n_max + k0 + u] = cn[u];
        }
      }
    }
    __syncthreads();
    // z~ = y - (y Z^T) Z (eq. rsvd_za) by one half of the threads, the next
    // sample against the rows accepted before this step by the other
    const double *cf = coef + half * n_max;
    double *row = half ? yn : y;
    for (int a = ht; a < n_vir; a += HALF) {
      double v = 0.0;
      const double *zc = Zb + a;
#pragma unroll 8
      for (int k = 0; k < s; ++k) v += cf[k] * zc[(int64_t)k * n_vir];
      row[a] = row[a] - v;
    }
    __syncthreads();
    // 1 / |z~| by every wave
    double n2[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      double q = 0.0;
      for (int a = 64 * u + lane; a < n_vir; a += 256) q += y[a] * y[a];
      n2[u] = rf_wave_sum(q);
    }
    const double inv = 1.0 / sqrt(((n2[0] + n2[1]) + n2[2]) + n2[3]);
    for (int a = threadIdx.x; a < n_vir; a += RF_THREADS) z[a] = y[a] * inv;
    // the accepted direction out of every row that pends next
    for (int j = wv; j < r; j += NW) {
      double *yj = Yb + (int64_t)(s + 1 + j) * n_vir;
      double c = 0.0;
      for (int a = lane; a < n_vir; a += 64) c += yj[a] * (y[a] * inv);
      c = rf_wave_sum(c);
      double q = 0.0;
      for (int a = lane; a < n_vir; a += 64) {
        const double v = yj[a] - c * (y[a] * inv);
        yj[a] = v;
        q += v * v;
      }
      q = rf_wave_sum(q);
      if (lane == 0) nrm[j] = sqrt(q);
    }
    __syncthreads();
    ++s;
  }
  for (int64_t e = (int64_t)s * n_vir + threadIdx.x; e < (int64_t)n_max * n_vir; e += RF_THREADS)
    Zb[e] = 0.0;
  if (threadIdx.x == 0) rows[b] = s;
}

hipError_t launch_range_finder(double *Y, double *Z, int32_t *rows, int nb, int r, int n_max,
                               int n_vir, double thr, hipStream_t s) {
  if (nb <= 0) return hipSuccess;
  const size_t smem = sizeof(double) * (2 * (size_t)n_max + r);
  hipLaunchKernelGGL(range_finder_kernel, dim3(nb), dim3(RF_THREADS), smem, s, Y, Z, rows, r,
                     n_max, n_vir, thr);
  return hipGetLastError();
}

// evals: [nb][D] eigenvalues of T~ T~^T ascending (sentinel beyond rows[b]);
// Qr: [nb][n_max][n_vir], row k = eigenvector k applied to Z (ascending
// order).  Output: Q_out rows of LMO i0 + b at (i0 + b) * n_max, decreasing
// w, only w >= l_osv, zero rows after; w_out likewise; n_osv[i0 + b].
__global__ __launch_bounds__(256) void rosv_finalize_kernel(
    const double *__restrict__ evals, int D, const double *__restrict__ Qr,
    const int32_t *__restrict__ rows, int i0, int n_max, int n_vir, double l_osv,
    double *__restrict__ Q_out, double *__restrict__ w_out, int32_t *__restrict__ n_osv,
    int32_t *__restrict__ rows_out) {
  __shared__ int keep;
  const int b = blockIdx.x;
  const int s = rows[b];
  const double *ev = evals + (int64_t)b * D;
  if (threadIdx.x == 0) {
    int k = 0;
    for (int j = s - 1; j >= 0; --j) {
      const double w = sqrt(fmax(ev[j], 0.0));
      if (w >= l_osv) ++k; else break;  // decreasing: the rest are smaller
    }
    keep = k;
    n_osv[i0 + b] = k;
    rows_out[i0 + b] = s;
  }
  __syncthreads();
  const int k = keep;
  double *qo = Q_out + (int64_t)(i0 + b) * n_max * n_vir;
  const double *qr = Qr + (int64_t)b * n_max * n_vir;
  for (int64_t e = threadIdx.x; e < (int64_t)n_max * n_vir; e += 256) {
    const int mu = (int)(e / n_vir);
    const int a = (int)(e - (int64_t)mu * n_vir);
    qo[e] = mu < k ? qr[(int64_t)(s - 1 - mu) * n_vir + a] : 0.0;
  }
  for (int mu = threadIdx.x; mu < n_max; mu += 256)
    w_out[(int64_t)(i0 + b) * n_max + mu] = mu < k ? sqrt(fmax(ev[s - 1 - mu], 0.0)) : 0.0;
}

hipError_t launch_rosv_finalize(const double *evals, int D, const double *Qr,
                                const int32_t *rows, int i0, int nb, int n_max, int n_vir,
                                double l_osv, double *Q_out, double *w_out, int32_t *n_osv,
                                int32_t *rows_out, hipStream_t s) {
  if (nb <= 0) return hipSuccess;
  hipLaunchKernelGGL(rosv_finalize_kernel, dim3(nb), dim3(256), 0, s, evals, D, Qr, rows, i0,
                     n_max, n_vir, l_osv, Q_out, w_out, n_osv, rows_out);
  return hipGetLastError();
}

}  // namespace mbe3
