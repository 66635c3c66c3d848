// Occupied-orbital localization (the paper's section on occupied orbital
// localization: Alg. 2, eq. loc_theta): Pipek-Mezey with Jacobi sweeps on
// Loewdin charges.
//
//   pm_charges_kernel  P^A_ij = sum_{alpha in A} C~_{alpha i} C~_{alpha j},
//                      stored P[(i n + j) n_atom + A] (atoms fastest, so a
//                      pair's three charge vectors and a row's update run
//                      along contiguous memory)
//   pm_step_kernel     one antidiagonal i + j = t of a sweep.  The algorithm
//                      walks the pairs i < j row by row; a pair's angle reads
//                      P_ij, P_ii and P_jj, which only rotations sharing i or
//                      j change, so (i, j) has to follow (i, j - 1) and
//                      (i - 1, j) alone and every pair of one antidiagonal can
//                      turn at once, from the angles and charges the
//                      row-by-row walk would have at that point.  A sweep is
//                      2 n - 3 dependent steps instead of n (n - 1) / 2.
// Per pair: a_ij and b_ij reduced over the atoms, 4 theta = atan2(b, -a), the
// increment sqrt(a^2 + b^2)(1 - cos 4 theta), then the rotation of the columns
// i, j of U and of the first and the second orbital index of every P^A; sweeps
// repeat while the last sweep's summed increment exceeds l_loc.
// Sums run in a fixed order, so the result is reproducible bit for bit.
#include "internal.hpp"

namespace mbe3 {

__global__ __launch_bounds__(256) void pm_charges_kernel(const double *__restrict__ C,
                                                         const int32_t *__restrict__ ao_off,
                                                         int n, int na, double *__restrict__ P) {
  const int64_t total = (int64_t)n * n * na;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int A = (int)(e % na);
    const int64_t ij = e / na;
    const int i = (int)(ij / n), j = (int)(ij - (int64_t)i * n);
    double acc = 0.0;
    for (int al = ao_off[A]; al < ao_off[A + 1]; ++al)
      acc += C[(int64_t)al * n + i] * C[(int64_t)al * n + j];
    P[e] = acc;
  }
}

hipError_t launch_pm_charges(const double *C, const int32_t *ao_off, int n, int na, double *P,
                             hipStream_t s) {
  const int64_t total = (int64_t)n * n * na;
  if (total <= 0) return hipSuccess;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(pm_charges_kernel, dim3((unsigned)blocks), dim3(256), 0, s, C, ao_off, n,
                     na, P);
  return hipGetLastError();
}

// Orbitals of step t (pairs i + j = t, i < j) as groups: first the pairs
// (lo + g, t - lo - g), then the orbitals without a partner in this step.
struct PmStep {
  int t, n, lo, npair;
};
static inline PmStep pm_step(int t, int n) {
  PmStep st;
  st.t = t;
  st.n = n;
  st.lo = t >= n ? t - n + 1 : 0;
  st.npair = (t - 1) / 2 - st.lo + 1;
  return st;
}
__device__ __forceinline__ void pm_group(const PmStep &st, int g, int &i, int &j) {
  j = -1;
  if (g < st.npair) {
    i = st.lo + g;
    j = st.t - i;
    return;
  }
  const int s = g - st.npair;  // below lo, above t - lo, or the middle t / 2
  if (s < st.lo) {
    i = s;
  } else {
    i = st.t - st.lo + 1 + (s - st.lo);
    if (i >= st.n) i = st.t >> 1;
  }
}

struct PmRot {
  double c, s;
  int32_t rot, pad_;
};

// Lanes that form one angle together.
static constexpr int PM_AL = 32;
static constexpr int PM_CB = 256 / PM_AL - 1;  // column groups of one workgroup

// Angle of the pair (i, j) on a group of PM_AL lanes (lane l of it): every
// lane returns it; *inc gets the increment (-1 for a pair that is not
// rotated).  cos and sin of theta by two half-angle steps from cos 4 theta =
// -a / h, sin 4 theta = b / h, each taken from the larger of the two, instead of
// the chain of atan2, sin and cos (a fifth of a step).  The charges of 32 localized
// orbitals are off by 3.6e-17 (rms of eight problems) against 3.3e-17 with those.
// Vanishing, huge and non-finite a, b take the library functions.
__device__ __forceinline__ PmRot pm_angle(const double *P, int n, int na, int i, int j, int l,
                                          double *inc) {
  const double *pij = P + ((int64_t)i * n + j) * na;
  const double *pii = P + ((int64_t)i * n + i) * na;
  const double *pjj = P + ((int64_t)j * n + j) * na;
  double a = 0.0, b = 0.0;
#pragma unroll 4
  for (int A = l; A < na; A += PM_AL) {
    const double x = pij[A], d = pii[A] - pjj[A];
    a += x * x - 0.25 * d * d;
    b += x * d;
  }
  for (int o = PM_AL / 2; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
  }
  PmRot r;
  r.pad_ = 0;
  const double h = sqrt(a * a + b * b);
  double gain;
  if (h > 1e-140 && h < 1e140) {
    const double c4 = -a / h, s4 = b / h;
    double c2, s2;  // cos 2 theta >= 0
    if (c4 >= 0.0) {
      c2 = sqrt(0.5 + 0.5 * c4);
      s2 = 0.5 * s4 / c2;
      gain = b * b / (h - a);  // h (1 - c4) without the cancellation
    } else {
      s2 = copysign(sqrt(0.5 - 0.5 * c4), b);
      c2 = 0.5 * s4 / s2;
      gain = h + a;
    }
    r.c = sqrt(0.5 + 0.5 * c2);
    r.s = 0.5 * s2 / r.c;
    // a root of 1/2 + c2/2 just below 1 is rounded down: on average c^2 + s^2 is a
    // third of an ulp short at small angles, and columns of U shrink (9e-15 after
    // five sweeps of 160 orbitals).  1 - s^2 / (1 + c) has no such bias.
    r.c = 1.0 - r.s * r.s / (1.0 + r.c);
  } else {
    const double th = 0.25 * atan2(b, -a);
    r.s = sin(th);
    r.c = cos(th);
    gain = h * (1.0 - cos(4.0 * th));
  }
  r.rot = fabs(r.s) >= 1e-10;
  *inc = r.rot ? gain : -1.0;
  return r;
}

// Workgroup (x, y): row group x, column groups [PM_CB y, PM_CB y + PM_CB).
// Reads the charges from Pin and writes the rotated blocks to Pout.  With ang
// == null Pin and Pout are two buffers and every workgroup forms the angles of
// its own rows and columns from Pin, so that one launch is one step; else Pin
// == Pout and pm_angle_kernel ran before.  Each element is read and written by
// one thread, the first of its blocks ahead of the angles.  A step moves all of
// P: bound by the launch and two chains of loads, then by memory.  Measured
// over a whole localization (5 sweeps) against one workgroup walking the pairs
// one by one: 7.7 ms for 213 ms (96 orbitals, 72 atoms; 7.6 us a step), 25.5 ms
// for 1377 ms (160, 120), 1.0 ms for 3.4 ms (24, 18), 0.61 ms for 0.86 ms (12, 9).
__global__ __launch_bounds__(256) void pm_step_kernel(const double *Pin, double *Pout,
                                                      double *__restrict__ U, PmStep st, int na,
                                                      const PmRot *__restrict__ ang,
                                                      double *__restrict__ inc) {
  __shared__ PmRot rt[PM_CB + 1];
  const int tid = threadIdx.x, n = st.n;
  const int ng = n - st.npair;
  const int b0 = blockIdx.y * PM_CB, nb = min(PM_CB, ng - b0);
  int i, j;
  pm_group(st, blockIdx.x, i, j);
  struct Item {
    int bg;  // column group, -1: none
    int64_t ik, il, jk, jl;
    double xik, xil, xjk, xjl;
  };
  auto fetch = [&](int e) {
    Item t;
    t.bg = -1;
    if (e >= nb * na) return t;
    const int bg = e / na, A = e - bg * na;
    int k, l;
    pm_group(st, b0 + bg, k, l);
    t.bg = bg;
    t.ik = ((int64_t)i * n + k) * na + A;
    t.il = l < 0 ? -1 : ((int64_t)i * n + l) * na + A;
    t.jk = j < 0 ? -1 : ((int64_t)j * n + k) * na + A;
    t.jl = j < 0 || l < 0 ? -1 : ((int64_t)j * n + l) * na + A;
    t.xik = Pin[t.ik];
    t.xil = t.il < 0 ? 0.0 : Pin[t.il];
    t.xjk = t.jk < 0 ? 0.0 : Pin[t.jk];
    t.xjl = t.jl < 0 ? 0.0 : Pin[t.jl];
    return t;
  };
  Item cur = fetch(tid), nxt = fetch(tid + 256);
  {
    const int u = tid / PM_AL, l = tid % PM_AL;  // u = 0: own rows, 1 + b: column group
    if (u <= nb) {
      const int g = u == 0 ? (int)blockIdx.x : b0 + u - 1;
      PmRot r = {1.0, 0.0, 0, 0};
      if (g < st.npair) {
        if (ang) {
          r = ang[g];
        } else {
          int gi, gj;
          double v;
          pm_group(st, g, gi, gj);
          r = pm_angle(Pin, n, na, gi, gj, l, &v);
          if (u == 0 && l == 0 && blockIdx.y == 0) inc[(int64_t)gi * n + gj] = v;
        }
      }
      if (l == 0) rt[u] = r;
    }
  }
  __syncthreads();
  const PmRot ra = rt[0];
  if (blockIdx.y == 0 && ra.rot) {  // columns i, j of U
    for (int k = tid; k < n; k += 256) {
      const double ui = U[(int64_t)k * n + i], uj = U[(int64_t)k * n + j];
      U[(int64_t)k * n + i] = ra.c * ui + ra.s * uj;
      U[(int64_t)k * n + j] = ra.c * uj - ra.s * ui;
    }
  }
  for (int e = tid; cur.bg >= 0; e += 256) {
    const PmRot rb = rt[cur.bg + 1];
    double xik = cur.xik, xil = cur.xil, xjk = cur.xjk, xjl = cur.xjl;
    if (ra.rot) {  // first index
      const double x = xik, y = xjk, z = xil, w = xjl;
      xik = ra.c * x + ra.s * y;
      xjk = ra.c * y - ra.s * x;
      xil = ra.c * z + ra.s * w;
      xjl = ra.c * w - ra.s * z;
    }
    if (rb.rot) {  // second index
      const double x = xik, y = xil, z = xjk, w = xjl;
      xik = rb.c * x + rb.s * y;
      xil = rb.c * y - rb.s * x;
      xjk = rb.c * z + rb.s * w;
      xjl = rb.c * w - rb.s * z;
    }
    Pout[cur.ik] = xik;
    if (cur.il >= 0) Pout[cur.il] = xil;
    if (cur.jk >= 0) Pout[cur.jk] = xjk;
    if (cur.jl >= 0) Pout[cur.jl] = xjl;
    cur = nxt;
    nxt = fetch(e + 512);
  }
}

// Angles of one step's pairs (PM_AL lanes each) for the in-place form.
__global__ __launch_bounds__(256) void pm_angle_kernel(const double *__restrict__ P, PmStep st,
                                                       int na, PmRot *__restrict__ ang,
                                                       double *__restrict__ inc) {
  const int g = (blockIdx.x * 256 + threadIdx.x) / PM_AL, l = threadIdx.x % PM_AL;
  if (g >= st.npair) return;
  int i, j;
  double v;
  pm_group(st, g, i, j);
  const PmRot r = pm_angle(P, st.n, na, i, j, l, &v);
  if (l == 0) {
    ang[g] = r;
    inc[(int64_t)i * st.n + j] = v;
  }
}

// rec[0] = the sweep's summed increment, rec[1] = rotations applied in it.
__global__ __launch_bounds__(1024) void pm_sweep_kernel(const double *__restrict__ inc, int n,
                                                        double *__restrict__ rec) {
  __shared__ double rs[16], rc[16];
  double s = 0.0, c = 0.0;
#pragma unroll 4
  for (int64_t e = threadIdx.x; e < (int64_t)n * n; e += 1024) {
    const double v = inc[e];
    if (e / n < e % n && v != -1.0) {
      s += v;
      c += 1.0;
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    s += __shfl_xor(s, o, 64);
    c += __shfl_xor(c, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    rs[threadIdx.x >> 6] = s;
    rc[threadIdx.x >> 6] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    s = c = 0.0;
    for (int w = 0; w < 16; ++w) {
      s += rs[w];
      c += rc[w];
    }
    rec[0] = s;
    rec[1] = c;
  }
}

__global__ __launch_bounds__(256) void pm_identity_kernel(double *__restrict__ U, int n) {
  const int64_t e = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (e < (int64_t)n * n) U[e] = e / n == e % n ? 1.0 : 0.0;
}

hipError_t launch_pm_identity(double *U, int n, hipStream_t s) {
  hipLaunchKernelGGL(pm_identity_kernel, dim3((unsigned)(((int64_t)n * n + 255) / 256)),
                     dim3(256), 0, s, U, n);
  return hipGetLastError();
}

int64_t pm_ws_doubles(int n) {  // increments, then angles (3 doubles each)
  return (int64_t)n * n + 3LL * (n / 2 + 1);
}

// Two buffers save the launch of the angles; in place a step touches half the
// memory.  Measured per step, two buffers against in place: 8.7 and 9.6 us at
// 5 MiB of charges, 16.5 and 17.3 at 23 MiB, 38.3 and 37.0 at 88 MiB, 111 and
// 77 at 220 MiB.
bool pm_two_buffers(int n, int na) { return (int64_t)n * n * na * 8 <= 64LL << 20; }

hipError_t launch_pm_sweep(double **P, double **P2, double *U, int n, int na, double *ws,
                           double *rec, hipStream_t s) {
  static_assert(sizeof(PmRot) == 24, "three doubles per angle");
  double *inc = ws;
  PmRot *ang = (PmRot *)(ws + (int64_t)n * n);
  for (int t = 1; t <= 2 * n - 3; ++t) {
    const PmStep st = pm_step(t, n);
    const int ng = n - st.npair;
    const dim3 grid(ng, (ng + PM_CB - 1) / PM_CB);
    if (*P2) {
      hipLaunchKernelGGL(pm_step_kernel, grid, dim3(256), 0, s, (const double *)*P, *P2, U, st,
                         na, (const PmRot *)nullptr, inc);
      double *x = *P;
      *P = *P2;
      *P2 = x;
    } else {
      hipLaunchKernelGGL(pm_angle_kernel, dim3((st.npair * PM_AL + 255) / 256), dim3(256), 0, s,
                         (const double *)*P, st, na, ang, inc);
      hipLaunchKernelGGL(pm_step_kernel, grid, dim3(256), 0, s, (const double *)*P, *P, U, st,
                         na, (const PmRot *)ang, inc);
    }
  }
  hipLaunchKernelGGL(pm_sweep_kernel, dim3(1), dim3(1024), 0, s, (const double *)inc, n, rec);
  return hipGetLastError();
}

}  // namespace mbe3
