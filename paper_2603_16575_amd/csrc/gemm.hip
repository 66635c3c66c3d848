// Grouped FP64 GEMM engine on the CDNA matrix cores (v_mfma_f64_16x16x4): a
// general kernel, and gemm_tiles_kernel for the lists that gemm_list_form names
// (all but those with a single row, column or step along a contiguous dimension).
//
// One workgroup (4 wave64) computes one BM x BN tile of one task.  Operand
// tiles of depth 16 are staged through two LDS buffers with coalesced global
// reads (k-contiguous or m/n-contiguous depending on the transpose flags):
// the next tile is loaded into registers while the current one feeds the
// matrix cores, then stored to the other buffer, one barrier per step.  LDS
// tiles are k-major so each MFMA operand read is 16 consecutive doubles.
// Stored rows of either operand may be gathered through an index list (rows
// of A = M index when A is not transposed, K index when it is; rows of B = K
// index when B is not transposed, N index when it is), which lets one task
// project a slab onto the OSVs of all neighbours of an orbital, form a
// 4-block pair K from two scattered row blocks, or contract gradient blocks
// of many pairs in one K-concatenated product.  A task may also store C^T
// (the coupling blocks are needed in both orientations).
#include "internal.hpp"

namespace mbe3 {

typedef double d4 __attribute__((ext_vector_type(4)));

template <int BM, int BN>
__global__ __launch_bounds__(256, 2) void gemm_tasks_kernel(
    const GemmTask *__restrict__ tasks, int n_tasks, GemmBases bases) {
  constexpr int BK = 16;
  // pitch = BM + 16: the four k-rows an MFMA read touches (lane / 16) start
  // 2 PA = 32 (mod 64) banks apart, so each half-wave reads distinct banks
  constexpr int PA = BM + 16;
  constexpr int PB = BN + 16;
  __shared__ double As[2][BK * PA];
  __shared__ double Bs[2][BK * PB];

  const int64_t tile = blockIdx.x;
  int lo = 0, hi = n_tasks - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tasks[mid].tile_begin <= tile) lo = mid; else hi = mid - 1;
  }
  const GemmTask t = tasks[lo];
  const int64_t local = tile - t.tile_begin;
  const int m0 = (int)(local / t.tiles_n) * BM;
  const int n0 = (int)(local % t.tiles_n) * BN;
  const double *__restrict__ A = bases.p[t.a_buf] + t.a_off;
  const double *__restrict__ B = bases.p[t.b_buf] + t.b_off;
  double *__restrict__ C = bases.p[t.c_buf] + t.c_off;
  double *__restrict__ CT = t.ct_off >= 0 ? bases.p[t.c_buf] + t.ct_off : nullptr;
  const int32_t *__restrict__ rows = bases.rows;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  constexpr int WM = BM / 2, WN = BN / 2;
  constexpr int TM = WM / 16, TN = WN / 16;
  const int wr = wave >> 1, wc = wave & 1;

  d4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

  // A / B elements per thread: a tile of BM x 16 split evenly when that
  // gives a power of two per thread, else 8 per thread on the first
  // BM * 16 / 8 threads (the 96-wide tiles: 192 of 256 threads load)
  constexpr int EA0 = BM * BK / 256, EB0 = BN * BK / 256;
  constexpr int EA = (BK % EA0 == 0) ? EA0 : 8;
  constexpr int EB = (BK % EB0 == 0) ? EB0 : 8;
  const bool a_act = tid < BM * BK / EA;
  const bool b_act = tid < BN * BK / EB;

  // Per-thread source positions.  k-contiguous A (transA = 0): EA consecutive
  // k of one row; m-contiguous A (transA = 1): EA consecutive m of one k row.
  // B likewise.  Gathered rows are resolved per k-row as they come.
  const int a_tpr = BK / EA;
  const int a_r = tid / a_tpr, a_k = (tid % a_tpr) * EA;
  int64_t a_row = -1;
  if (a_act && !t.transA && m0 + a_r < t.M)
    a_row = (t.a_rows >= 0) ? rows[t.a_rows + m0 + a_r] : (m0 + a_r);
  const int a_tpk = BM / EA;
  const int a_kk = tid / a_tpk, a_mm = (tid % a_tpk) * EA;
  const int b_tpr = BK / EB;
  const int b_r = tid / b_tpr, b_k = (tid % b_tpr) * EB;
  int64_t b_row = -1;
  if (b_act && t.transB && n0 + b_r < t.N)
    b_row = (t.b_rows >= 0) ? rows[t.b_rows + n0 + b_r] : (n0 + b_r);
  const int b_tpk = BN / EB;
  const int b_kk = tid / b_tpk, b_nn = (tid % b_tpk) * EB;

  double ra[EA], rb[EB];  // the next tile, in flight during the products
#define MBE3_GEMM_LOAD(K0)                                                     \
  do {                                                                         \
    if (!t.transA) {                                                           \
      _Pragma("unroll") for (int e = 0; e < EA; ++e) {                         \
        const int k = (K0) + a_k + e;                                          \
        ra[e] = (a_row >= 0 && k < t.K) ? A[a_row * (int64_t)t.lda + k] : 0.0; \
      }                                                                        \
    } else {                                                                   \
      const int k = (K0) + a_kk;                                               \
      const int64_t krow = k < t.K ? (t.a_rows >= 0 ? rows[t.a_rows + k] : k) : 0; \
      _Pragma("unroll") for (int e = 0; e < EA; ++e) {                         \
        const int m = m0 + a_mm + e;                                           \
        ra[e] = (a_act && m < t.M && k < t.K) ? A[krow * t.lda + m] : 0.0;     \
      }                                                                        \
    }                                                                          \
    if (!t.transB) {                                                           \
      const int k = (K0) + b_kk;                                               \
      const int64_t krow = k < t.K ? (t.b_rows >= 0 ? rows[t.b_rows + k] : k) : 0; \
      _Pragma("unroll") for (int e = 0; e < EB; ++e) {                         \
        const int n = n0 + b_nn + e;                                           \
        rb[e] = (b_act && n < t.N && k < t.K) ? B[krow * t.ldb + n] : 0.0;     \
      }                                                                        \
    } else {                                                                   \
      _Pragma("unroll") for (int e = 0; e < EB; ++e) {                         \
        const int k = (K0) + b_k + e;                                          \
        rb[e] = (b_row >= 0 && k < t.K) ? B[b_row * (int64_t)t.ldb + k] : 0.0; \
      }                                                                        \
    }                                                                          \
  } while (0)
#define MBE3_GEMM_STORE(BUF)                                                   \
  do {                                                                         \
    double *as_ = As[BUF];                                                     \
    double *bs_ = Bs[BUF];                                                     \
    if (!a_act) {                                                              \
    } else if (!t.transA) {                                                    \
      _Pragma("unroll") for (int e = 0; e < EA; ++e) as_[(a_k + e) * PA + a_r] = ra[e]; \
    } else {                                                                   \
      _Pragma("unroll") for (int e = 0; e < EA; ++e) as_[a_kk * PA + a_mm + e] = ra[e]; \
    }                                                                          \
    if (!b_act) {                                                              \
    } else if (!t.transB) {                                                    \
      _Pragma("unroll") for (int e = 0; e < EB; ++e) bs_[b_kk * PB + b_nn + e] = rb[e]; \
    } else {                                                                   \
      _Pragma("unroll") for (int e = 0; e < EB; ++e) bs_[(b_k + e) * PB + b_r] = rb[e]; \
    }                                                                          \
  } while (0)

  MBE3_GEMM_LOAD(0);
  MBE3_GEMM_STORE(0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < t.K; k0 += BK) {
    const bool more = k0 + BK < t.K;
    if (more) MBE3_GEMM_LOAD(k0 + BK);
    const double *as = As[buf];
    const double *bs = Bs[buf];
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      const int kr = kk + (lane >> 4);
      double a[TM], b[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) a[i] = as[kr * PA + wr * WM + i * 16 + (lane & 15)];
#pragma unroll
      for (int j = 0; j < TN; ++j) b[j] = bs[kr * PB + wc * WN + j * 16 + (lane & 15)];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    // the other buffer was last read before the previous barrier
    if (more) MBE3_GEMM_STORE(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
#undef MBE3_GEMM_LOAD
#undef MBE3_GEMM_STORE

  // ---- epilogue: D layout of v_mfma_f64_16x16x4: register v of lane l holds
  //      row (l / 16) + 4 v, column l % 16
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + wc * WN + j * 16 + (lane & 15);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + wr * WM + i * 16 + (lane >> 4) + 4 * v;
        if (m < t.M && n < t.N) {
          double *c = C + (int64_t)m * t.ldc + n;
          double r = t.alpha * acc[i][j][v];
          if (t.beta != 0.0) r += t.beta * *c;
          *c = r;
          if (CT) CT[(int64_t)n * t.ldct + m] = r;
        }
      }
    }
}

// ---------------------------------------------------------------------------
// The same products for lists whose tasks agree on their transpose flags and
// have at least two elements along the contiguous dimension of either operand
// (gemm_list_form): 16-byte loads and 16-byte LDS stores.
//
// An operand tile (BD x 16) reaches the thread block in 16-byte chunks, in one
// of two forms fixed at compile time.
//   rows (K contiguous): 8 chunks per row, kept row by row in LDS, chunk c of
//     row r at place c ^ (r & 7), so that the 16 rows x 4 k's of an MFMA operand
//     read fall on all banks evenly;
//   k-major (M / N contiguous): BD / 2 chunks per k, chunk c of row k at place
//     c ^ (8 (k & 1)): the two k's of a half-wave's read then lie on different
//     halves of the banks, without a padded pitch.
// Every chunk is loaded from an address inside its operand, at 8-byte alignment:
// one that would reach past the end of its row starts one element earlier and is
// shifted, one past K is zeroed (the last step only).  Rows past M or N repeat
// the tile's first one and are not stored.  Each output sums over k in the order
// of the general kernel, so the results are the same bit for bit.
// Bound: matrix cores at the projection's 128 x 128 tiles (what is left is the
// load and store part of a step, which the second workgroup of the CU covers);
// the general kernel spent 16 loads, 16 stores and their guards on what takes 8
// and 8 here.  Measured against it: projection of 48 orbitals, 2432 x 7040 slabs,
// 41.6 ms for 45.9 ms (58.7 TF/s; a 8192^3 library product reaches 72), their pair
// K 3.59 ms for 4.94 ms, a 160-orbital step's trimer blocks 16.5 ms for 20.5 ms,
// its pair K 2.75 ms for 3.55 ms, the gradient's products 35.0 ms for 38.4 ms.
// ---------------------------------------------------------------------------
typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

template <int BD, bool KMAJOR>
struct TileLoader {
  static constexpr int NCH = BD / 32;  // chunks per thread
  const double *base;
  const int32_t *gather;  // k-major, gathered: row index of k; else null
  const double *ptr[NCH];  // rows: the chunk's row; k-major: its column
  int ld, K, c2;           // c2: rows: first k of the thread's chunks
  int32_t krow[NCH];       // k-major, gathered: rows of the next step's k's
  bool shift[NCH];         // k-major: the row's odd last element
  d2 v[NCH];

  // dim: rows of the operand along M / N; x0: first of the tile
  __device__ __forceinline__ void init(const double *b, const int32_t *rows, int rows_off,
                                       int ld_, int K_, int dim, int x0, int tid) {
    base = b;
    ld = ld_;
    K = K_;
    gather = KMAJOR && rows_off >= 0 ? rows + rows_off : nullptr;
    c2 = 2 * (tid & 7);
#pragma unroll
    for (int u = 0; u < NCH; ++u) {
      if (KMAJOR) {
        const int c = x0 + 2 * ((tid + 256 * u) % (BD / 2));
        ptr[u] = base + (c + 1 < dim ? c : c < dim ? c - 1 : x0 + 1 < dim ? x0 : dim - 2);
        shift[u] = c + 1 == dim;
      } else {
        int r = x0 + (tid >> 3) + 32 * u;
        r = r < dim ? r : x0;
        ptr[u] = base + (int64_t)(rows_off >= 0 ? rows[rows_off + r] : r) * ld;
        shift[u] = false;
      }
      krow[u] = 0;
    }
    if (gather) fetch_rows(0, tid);
  }
  __device__ __forceinline__ int k_of(int u, int tid) const { return (tid + 256 * u) / (BD / 2); }
  __device__ __forceinline__ void fetch_rows(int k0, int tid) {
#pragma unroll
    for (int u = 0; u < NCH; ++u) {
      const int k = k0 + k_of(u, tid);
      krow[u] = gather[k < K ? k : K - 1];
    }
  }
  __device__ __forceinline__ void load(int k0, int tid) {
    if (KMAJOR) {
#pragma unroll
      for (int u = 0; u < NCH; ++u) {
        const int k = k0 + k_of(u, tid);
        const int64_t row = gather ? krow[u] : (k < K ? k : K - 1);
        v[u] = *(const d2u *)(ptr[u] + row * ld);
      }
      if (gather && k0 + 16 < K) fetch_rows(k0 + 16, tid);
    } else {
      const int k = k0 + c2;
      const int64_t o = k + 1 < K ? k : K - 2;
#pragma unroll
      for (int u = 0; u < NCH; ++u) v[u] = *(const d2u *)(ptr[u] + o);
    }
  }
  __device__ __forceinline__ void store(double *l, int k0, int tid) {
#pragma unroll
    for (int u = 0; u < NCH; ++u) {
      d2 x = v[u];
      if (KMAJOR) {
        const int e = tid + 256 * u, k = e / (BD / 2), c = e % (BD / 2);
        if (shift[u]) x = d2{x.y, 0.0};
        if (k0 + k >= K) x = d2{0.0, 0.0};
        *(d2 *)(l + k * BD + 2 * (c ^ ((k & 1) << 3))) = x;
      } else {
        if (k0 + c2 + 1 >= K) x = k0 + c2 < K ? d2{x.y, 0.0} : d2{0.0, 0.0};
        const int r = (tid >> 3) + 32 * u;
        *(d2 *)(l + r * 16 + 2 * ((tid & 7) ^ (r & 7))) = x;
      }
    }
  }
};

// Operand reads: element (x, k) of the tile, x = 16 b + l16, k = kk + lq (b, kk
// compile-time apart from the wave's first block).
template <int BD, bool KMAJOR, int NB>
struct TileReader {
  int o0, o1;  // k-major: even / odd blocks; rows: the place at kk = 0
  __device__ __forceinline__ void init(int b0, int l16, int lq) {
    if (KMAJOR) {
      const int s = (lq & 1) << 4;
      const int o = lq * BD + b0 * 16 + l16;
      o0 = o + (b0 & 1 ? -s : s);
      o1 = o + (b0 & 1 ? s : -s);
    } else {
      o0 = (b0 * 16 + l16) * 16 + 2 * ((lq >> 1) ^ (l16 & 7)) + (lq & 1);
      o1 = 0;
    }
  }
  __device__ __forceinline__ void read(const double *l, int kk, double *x) const {
    if (KMAJOR) {
#pragma unroll
      for (int b = 0; b < NB; ++b) x[b] = l[(b & 1 ? o1 : o0) + kk * BD + b * 16];
    } else {
      const int o = o0 ^ kk;  // places kk / 2 on: bits 1.. of the element offset
#pragma unroll
      for (int b = 0; b < NB; ++b) x[b] = l[o + b * 256];
    }
  }
};

template <int BM, int BN, bool TA, bool TB>
__global__ __launch_bounds__(256, 2) void gemm_tiles_kernel(
    const GemmTask *__restrict__ tasks, int n_tasks, GemmBases bases) {
  __shared__ __align__(16) double As[2][BM * 16];
  __shared__ __align__(16) double Bs[2][BN * 16];
  const int64_t tile = blockIdx.x;
  int lo = 0, hi = n_tasks - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tasks[mid].tile_begin <= tile) lo = mid; else hi = mid - 1;
  }
  const GemmTask t = tasks[lo];
  const int local = (int)(tile - t.tile_begin);
  const int m0 = (local / t.tiles_n) * BM;
  const int n0 = (local % t.tiles_n) * BN;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, lq = lane >> 4;
  constexpr int TM = BM / 32, TN = BN / 32;  // 16-blocks per wave (2 x 2 waves)
  const int bm = (wave >> 1) * TM, bn = (wave & 1) * TN;

  TileLoader<BM, TA> la;
  TileLoader<BN, !TB> lb;
  la.init(bases.p[t.a_buf] + t.a_off, bases.rows, t.a_rows, t.lda, t.K, t.M, m0, tid);
  lb.init(bases.p[t.b_buf] + t.b_off, bases.rows, t.b_rows, t.ldb, t.K, t.N, n0, tid);
  TileReader<BM, TA, TM> ra;
  TileReader<BN, !TB, TN> rb;
  ra.init(bm, l16, lq);
  rb.init(bn, l16, lq);

  d4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};

  la.load(0, tid);
  lb.load(0, tid);
  la.store(As[0], 0, tid);
  lb.store(Bs[0], 0, tid);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < t.K; k0 += 16) {
    const bool more = k0 + 16 < t.K;
    if (more) {
      la.load(k0 + 16, tid);
      lb.load(k0 + 16, tid);
    }
#pragma unroll
    for (int kk = 0; kk < 16; kk += 4) {
      double a[TM], b[TN];
      ra.read(As[buf], kk, a);
      rb.read(Bs[buf], kk, b);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
    }
    // the other buffer was last read before the previous barrier
    if (more) {
      la.store(As[buf ^ 1], k0 + 16, tid);
      lb.store(Bs[buf ^ 1], k0 + 16, tid);
    }
    __syncthreads();
    buf ^= 1;
  }

  double *__restrict__ C = bases.p[t.c_buf] + t.c_off;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int n = n0 + (bn + j) * 16 + l16;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + (bm + i) * 16 + lq + 4 * v;
        double r = t.alpha * acc[i][j][v];
        if (m < t.M && n < t.N) {
          double *c = C + (int64_t)m * t.ldc + n;
          if (t.beta != 0.0) r += t.beta * *c;
          *c = r;
        }
        acc[i][j][v] = r;
      }
    }
  if (t.ct_off < 0) return;
  // C^T through LDS, one 16 x 16 block of a wave at a time, so that its rows
  // leave as 128-byte runs too (every wave is past its last operand read)
  double *__restrict__ CT = bases.p[t.c_buf] + t.ct_off;
  double *x = &As[0][0] + wave * (16 * 17 > BM * 8 ? BM * 8 : 16 * 17);
  constexpr bool FITS = BM * 8 >= 16 * 17;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      if (FITS) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int v = 0; v < 4; ++v) x[(lq + 4 * v) * 17 + l16] = acc[i][j][v];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + (bm + i) * 16 + (FITS ? l16 : lq + 4 * v);
        const int n = n0 + (bn + j) * 16 + (FITS ? lq + 4 * v : l16);
        const double r = FITS ? x[l16 * 17 + lq + 4 * v] : acc[i][j][v];
        if (m < t.M && n < t.N) CT[(int64_t)n * t.ldct + m] = r;
      }
      if (FITS) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
}

// Form of a task list: -1 general; else 2 transA + transB of all its tasks.
int gemm_list_form(const GemmTask *ts, int64_t n) {
  for (int64_t k = 0; k < n; ++k) {
    const GemmTask &t = ts[k];
    if (t.transA != ts[0].transA || t.transB != ts[0].transB) return -1;
    if ((t.transA ? t.M : t.K) < 2 || (t.transB ? t.K : t.N) < 2) return -1;
  }
  return n > 0 ? 2 * (ts[0].transA != 0) + (ts[0].transB != 0) : -1;
}

int gemm_tile_m(GemmShape shape) {
  switch (shape) {
    case GEMM_128x32:
    case GEMM_128x128: return 128;
    case GEMM_32x32:
    case GEMM_32x128: return 32;
    case GEMM_96x96: return 96;
    default: return 64;
  }
}

int gemm_tile_n(GemmShape shape) {
  switch (shape) {
    case GEMM_128x32:
    case GEMM_32x32: return 32;
    case GEMM_64x64: return 64;
    case GEMM_96x96: return 96;
    default: return 128;
  }
}

const char *gemm_shape_name(GemmShape shape) {
  switch (shape) {
    case GEMM_64x64: return "64x64";
    case GEMM_128x128: return "128x128";
    case GEMM_32x32: return "32x32";
    case GEMM_32x128: return "32x128";
    case GEMM_64x128: return "64x128";
    case GEMM_96x96: return "96x96";
    default: return "?";
  }
}

int64_t gemm_tile_count(const GemmTask &t, GemmShape shape) {
  const int bm = gemm_tile_m(shape), bn = gemm_tile_n(shape);
  return (int64_t)((t.M + bm - 1) / bm) * ((t.N + bn - 1) / bn);
}

template <int BM, int BN>
static hipError_t launch_shape(const GemmTask *ts, int n, dim3 grid, const GemmBases &b, int form,
                               hipStream_t s) {
  switch (form) {
    case 0:
      hipLaunchKernelGGL((gemm_tiles_kernel<BM, BN, false, false>), grid, dim3(256), 0, s, ts, n, b);
      break;
    case 1:
      hipLaunchKernelGGL((gemm_tiles_kernel<BM, BN, false, true>), grid, dim3(256), 0, s, ts, n, b);
      break;
    case 2:
      hipLaunchKernelGGL((gemm_tiles_kernel<BM, BN, true, false>), grid, dim3(256), 0, s, ts, n, b);
      break;
    case 3:
      hipLaunchKernelGGL((gemm_tiles_kernel<BM, BN, true, true>), grid, dim3(256), 0, s, ts, n, b);
      break;
    default:
      hipLaunchKernelGGL((gemm_tasks_kernel<BM, BN>), grid, dim3(256), 0, s, ts, n, b);
  }
  return hipGetLastError();
}

hipError_t launch_gemm_tasks(const GemmTask *d_tasks, int n_tasks,
                             int64_t n_tiles, const GemmBases &bases,
                             GemmShape shape, int form, hipStream_t s) {
  if (n_tasks <= 0 || n_tiles <= 0) return hipSuccess;
  if (n_tiles >= 1 << 24) return hipErrorInvalidValue;  // a grid past 2^32 threads wraps
  const dim3 grid((unsigned)n_tiles);
  switch (shape) {
    case GEMM_64x64: return launch_shape<64, 64>(d_tasks, n_tasks, grid, bases, form, s);
    case GEMM_128x128: return launch_shape<128, 128>(d_tasks, n_tasks, grid, bases, form, s);
    case GEMM_32x32: return launch_shape<32, 32>(d_tasks, n_tasks, grid, bases, form, s);
    case GEMM_32x128: return launch_shape<32, 128>(d_tasks, n_tasks, grid, bases, form, s);
    case GEMM_64x128: return launch_shape<64, 128>(d_tasks, n_tasks, grid, bases, form, s);
    case GEMM_96x96: return launch_shape<96, 96>(d_tasks, n_tasks, grid, bases, form, s);
    case GEMM_128x32: return launch_shape<128, 32>(d_tasks, n_tasks, grid, bases, form, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mbe3
