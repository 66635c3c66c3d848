// Fragment solver: the coupled residual equations of one 1-, 2- or 3-orbital
// fragment (eq. res_close restricted to the fragment, Algorithm 7) iterated
// to convergence inside one workgroup.
//
// Work is done in each pair's pseudo-canonical basis X (eq. prec_eig):
// T_pq = X Y X^T.  Then the pair's own Fock terms become diagonal,
//   X^T (F T S + S T F - f_pp S T S - f_qq S T S) X = -E~ o Y,
// and every coupling term f S_(t,s) T_s S_(s,t) becomes
//   f S~_(t,s) Y_s S~_(t,s)^T,   S~_(t,s) = X_t^T V_t^T V_s X_s,
// so one sweep is
//   R~_t = K~_t - E~_t o Y_t - sum_terms f S~ Y_s^(T) S~^T   (+ transpose for
//          diagonal pairs, whose two mirror terms are transposes),
//   converged if max |R~| < tol, else Y_t += R~_t / E~_t,
// which is the paper's update T += X (X^T R X / E~) X^T with the same
// iterates, without the per-sweep X transforms.  The Hylleraas energy
//   E_F = sum_t w_t <2 Y_t - Y_t^T, K~_t + R~_t>
// is accumulated in the same pass.
//
// Data flow of one term on the FP64 matrix cores (v_mfma_f64_16x16x4), with
// S~ stored as S~_(s,t) = S~'^T (D_s x D_t, row-major):
//   pass 1: for a 16-row block ib of R~_t a wave accumulates
//      W = Z^T = (Y_s^(T))^T S~'^T over 16-row panels m of Y_s^(T) and S~;
//   pass 2: the MFMA output layout (register v of lane l holds row l/16 + 4v,
//      column l%16) is exactly the A-operand layout of the second product for
//      the four k-steps kb*16 + 4v, so Z never leaves the registers and
//      R~_t[ib, :] += Z[ib, :] S~'^T reads the S~ resident in LDS.
// A wave works on one row block, whole or shared with other waves by source
// blocks kb (row_part): each then holds a partial R~_t[ib, :], added up through
// LDS once per target.  Before, the waves took whole blocks alone, and a SIMD
// with one block more than the others set the time of every product: 2 blocks
// against 1.25 on average at 80-wide targets.  The steps of a product that lie in
// the padding of the source are left out.
// Panels go global -> registers (prefetched one step ahead) -> LDS: the
// term's S~ panels land in a resident D_s x D_t block reused by pass 2 (which
// then needs no barrier and hides the next term's first load), the Y^(T)
// rows in two alternating 16-row buffers.  Only Y is kept in memory: a panel
// of Y^T (16 rows of it) is read as 16-column strips of Y's rows, kept as
// strips, and its operand read across them; the residual reads Y^T elements
// straight from Y, so each sweep writes its amplitudes once, coalesced.  The
// residual's inputs are fetched a block ahead with no load under a condition (a
// branch around one of them had every block wait for its own loads: a quarter of
// the solver).  LDS per workgroup is D_max^2 + 36 D_max doubles (18 D_max at
// D_max = 128, one Y buffer).  Up to 80-wide domains four waves work on a
// fragment, and two (80), three (64, 48) or four (32) fragments share a CU; above,
// eight waves and one fragment.  A diagonal pair's mirror terms f S~ Y S~^T and
// its transpose are formed once and symmetrised through LDS.
// What bounds it: about 45% of the wave time is products (matrix cores busy
// 40%), 15% the residual, the rest the panel steps and their barriers; 3 TB/s of
// S~ past L2.  Measured, all launches of a step: 88.8 ms for 119 ms at 160
// orbitals (D to 80), 116 ms for 135 ms at 96 orbitals of 24 - 64 OSVs (D to
// 128), 32 orbitals recorded with gradient 6.6 ms for 9.7 ms.
// Sweep 0 has T = 0, so R~ = K~ needs no product.  All pair blocks are zero
// padded to multiples of 16: no tile is masked.
#include <algorithm>
#include <type_traits>

#include "internal.hpp"

namespace mbe3 {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ d4 mfma_f64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Row pitch of a strip of 16 Y columns kept for a transposed source: 16 rows of
// it, read across, fall on distinct banks.
constexpr int YPITCH = 18;

// s_waitcnt immediate of vmcnt(0) alone (gfx9 encoding: expcnt and lgkmcnt
// at their maxima)
constexpr int WAIT_VMCNT0 = 0x0F70;

// A fragment's terms and slots as the workgroup reads them, staged in LDS at
// the start of each fragment: every panel step and residual block then reads
// its descriptors from LDS instead of chasing term -> slot -> dimension
// through global memory (each hop a full memory round trip on the critical
// path of the panel pipeline).
struct TermLds {
  const double *st;  // row-major S~_(src, target)
  double coef;       // f_occ[fx][fy]; 1 in the gradient pass
  int32_t src, dt, ds, ds0, trans, pad_;  // ds0: the source's unpadded dimension
};
struct SlotLds {
  int64_t kt_off, et_off;
  const double *gy;  // gradient pass: the amplitudes its terms read
  double fpq;  // f_pp + f_qq
  int32_t D, ysub, sym, wgt;  // sym: 1 diagonal, 2 diagonal with an unsymmetric K~
  int32_t tb, tx, te;  // the slot's terms of this launch in tc[], the first
                       // of them that couples two pairs of a trimer
  int64_t b0, b1;      // coupling sums of the slot (second one: diagonal
                       // slots of a trimer)
};

// Offset of the coupling sums of pair slot sl: on its first orbital (w = 0),
// its second (1), the pair itself (2).
__device__ __forceinline__ int64_t base_of(const SlotInfo *slots, const SlotInfo &sl, int w) {
  int64_t o = sl.base_off;
  if (w > 0) o += (int64_t)slots[sl.p].D * slots[sl.p].D;
  if (w > 1) o += (int64_t)slots[sl.q].D * slots[sl.q].D;
  return o;
}

// Sum / max of the per-wave partials r[0 .. N) as a fixed tree: the first
// half (the largest power of two below N) and the rest, recursively.
template <int N>
__device__ __forceinline__ double wave_tree_sum(const double *r) {
  if constexpr (N == 1) {
    return r[0];
  } else {
    constexpr int H = N > 4 ? 4 : (N > 2 ? 2 : 1);
    return wave_tree_sum<H>(r) + wave_tree_sum<N - H>(r + H);
  }
}
template <int N>
__device__ __forceinline__ double wave_tree_max(const double *r) {
  if constexpr (N == 1) {
    return r[0];
  } else {
    constexpr int H = N > 4 ? 4 : (N > 2 ? 2 : 1);
    return fmax(wave_tree_max<H>(r), wave_tree_max<N - H>(r + H));
  }
}

// Workgroup sum in a fixed order (wave shuffles, then the waves' tree).
template <int NW>
__device__ __forceinline__ double wg_sum(double v, double *red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  const double s = wave_tree_sum<NW>(red);
  __syncthreads();
  return s;
}

// Raw buffer loads of 16 bytes: lanes past num bytes read zero without a
// branch, and the panel's offset is one scalar.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const double *p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(p), 0, bytes, 0x00027000);
}
__device__ __forceinline__ d2 load_b128(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(d2, (u4)__builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}
// Volatile views of LDS: a load stays where it is written, ahead of the guarded
// product that uses it.
typedef __attribute__((address_space(3))) const volatile double lds_d;
__device__ __forceinline__ const lds_d *as_lds(const double *p) { return (const lds_d *)p; }
// A value all lanes share, in scalar registers.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform(int64_t v) {
  return (int64_t)(((uint64_t)(uint32_t)uniform((int)((uint64_t)v >> 32)) << 32) |
                   (uint32_t)uniform((int)v));
}
__device__ __forceinline__ double uniform(double v) {
  return __builtin_bit_cast(double, uniform(__builtin_bit_cast(int64_t, v)));
}
__device__ __forceinline__ const double *uniform(const double *p) {
  return (const double *)uniform((int64_t)p);
}
// Element o of a block in global memory (which a pointer made of scalars no
// longer says): scalar base, 32-bit offset.
typedef __attribute__((address_space(1))) double g_double;
__device__ __forceinline__ double at(const double *p, uint32_t o) {
  return *(const g_double *)((const char *)p + o * 8u);
}
__device__ __forceinline__ void put(double *p, uint32_t o, double v) {
  *(g_double *)((char *)p + o * 8u) = v;
}
constexpr int OOB = 0x7fff0000;  // past every block

// Elements of a register array, however many are used: an array of up to 16
// doubles would become one vector value, copied whole wherever one of its
// elements is written under a guard (up to 90 moves per matrix instruction at
// 64-wide domains).
constexpr int SPLIT = 9;

// Which 16-row block of a target with nT of them a wave works on, and which
// share of that block's source blocks: part of nparts, source blocks kb with kb
// mod nparts == part.  The waves of one block are first, first + stride, ...
// Waves w and w + 4 share a SIMD, so for eight waves every SIMD gets nT / 4 of
// a row's products (7 rows: 2): four rows go whole to waves 0 - 3, the rest is
// dealt to waves 4 - 7.  ib = -1: nothing to do.
struct RowPart {
  int ib, part, lg, first, stride;  // nparts = 1 << lg
};
template <int NW>
__device__ __forceinline__ RowPart row_part(int nT, int w) {
  if (NW == 8) {
    if (nT >= 7) return {w < nT ? w : -1, 0, 0, w, 1};
    if (nT == 4) return {w & 3, w >> 2, 1, w & 3, 4};
    if (nT == 1) return {0, w, 3, 0, 1};
    if (nT == 2) return {w >> 2, w & 3, 2, w & 4, 1};
    if (w < 4) return nT == 3 ? RowPart{0, w, 2, 0, 1} : RowPart{w, 0, 0, w, 1};
    if (nT == 5) return {4, w & 3, 2, 4, 1};
    return {(nT == 3 ? 1 : 4) + ((w & 2) >> 1), w & 1, 1, w & 6, 1};
  }
  if (nT >= 3) return {w < nT ? w : -1, 0, 0, w, 1};
  if (nT == 1) return {0, w, 2, 0, 1};
  return {w >> 1, w & 1, 1, w & 2, 1};
}
// The blocks < n of part of 1 << lg parts as a bit mask.
__device__ __forceinline__ uint32_t part_mask(int part, int lg, int n) {
  const uint32_t every = lg == 0 ? 0xffu : lg == 1 ? 0x55u : lg == 2 ? 0x11u : 1u;
  return (every << part) & ((1u << n) - 1u);
}

// MAXNT: largest number of 16-blocks per pair dimension (dmax / 16).
// MODE 0: solve.  MODE 1: solve and store each converged fragment's Y at
// FragDesc::yout (zero if it converged at T = 0) for the gradient pass.
// A warm-started trimer's first sweep reads the solutions of its pairs' own
// fragments, so two thirds of its terms (a pair and one of its orbitals) depend
// on the pair alone: MODE 3 forms those sums once per pair, over the warm
// store, and the trimers' first sweep adds them in its residual instead of
// forming them again in each of the pair's trimers (about 50; the planner leaves
// them out where it is less than two).  All solver launches of 160 orbitals with
// and without them: 88.6 and 100.4 ms, the sums 0.4 of it.
// MODE 2: the gradient pass alone, a separate launch over the same
// fragments: the terms [tb, tg) of each pair target are formed once more from
// the stored Y with unit coefficient and contracted with Y~ = 2Y - Y^T.  The
// coupling operator is symmetric, so a term's contraction equals its mirror's
// (source and target exchanged) up to the pair weights (an unsymmetric diagonal
// source is adapted to that), and 9 of a trimer's 18 terms are enough: of a pair and
// its orbital the pair's (the wider target, which leaves fewer waves without a row
// block), of two pairs one each way round the trimer.  Measured at 160 orbitals (90k
// fragments): 28.4 ms for 59.8 ms with every term.  Fragments that did not converge
// (iters < 0) are skipped.  Keeping the pass out of the solving launch keeps its
// registers out of the iterations.
template <int MAXNT, int MODE, int NW>
__global__ __launch_bounds__(64 * NW, MAXNT == 5 ? 2 : NW == 4 ? 3 : 1) void solve_kernel(SolveArgs a) {
  constexpr bool ST = MODE == 1, GP = MODE == 2, BASE = MODE == 3;
  extern __shared__ double lds[];
  constexpr int NTH = 64 * NW;                     // threads per workgroup
  constexpr int PFN = (8 * 16 * MAXNT + NTH - 1) / NTH;  // slots of a panel's S~ (or Y)
  constexpr bool DBY = MAXNT <= 7;                 // two Y panel buffers
  constexpr bool ROW2 = NW == 4 && MAXNT == 5;     // a fifth row block, shared
  constexpr int NR2 = ROW2 ? MAXNT : 1, NW2 = ROW2 ? 2 : 1;
  __shared__ double red_d[2 * NW];
  __shared__ int red_i[NW];
  __shared__ TermLds tc[MAX_FRAG_TERMS];
  __shared__ SlotLds sc[6];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = uniform(tid >> 6);  // uniform per wave
  const int l16 = lane & 15;
  const int lq = lane >> 4;
  // LDS: the term's whole S~ (D_s x D_t) stays resident for both passes; the
  // Y^(T) rows stream through two 16-row buffers.
  double *const Sl = lds;
  double *const yb0 = lds + (int64_t)a.dmax * a.dmax;
  double *const yb1 = DBY ? yb0 + YPITCH * a.dmax : yb0;

  double *scr = a.scratch + (int64_t)blockIdx.x * a.scratch_stride;
  const int64_t ny_cap = (a.scratch_stride - 2LL * a.dmax * a.dmax) / 4;
  double *const Y0 = scr;  // two buffers of ny_cap (current, next)

  d2 ps[SPLIT], py[SPLIT];  // next panel: S~ rows, Y^(T) rows (PFN used)

  for (int fi = blockIdx.x; fi < a.n_frag; fi += gridDim.x) {
    const FragDesc *__restrict__ fdp = a.frags + fi;
    const int f_nt = fdp->nt, f_frag = fdp->frag;
    const int f_tb = fdp->term_begin, f_te = fdp->term_end;
    int cur = 0;
    // amplitudes present: after a warm start from the solutions of the
    // fragment's own pairs (monomers, dimers), or after the first update
    bool hasY = false;
    if (GP && a.iters[f_frag] < 0) continue;  // uniform over the workgroup
    if (BASE && (f_nt != 3 || a.slots[fdp->slot[2]].base_off < 0)) continue;
    // stage the descriptors (the previous fragment's last reads of them came
    // before its closing barrier)
    if (tid < f_te - f_tb) {
      const Term t = a.terms[f_tb + tid];
      TermLds c;
      c.st = (t.st_buf ? a.st1 : a.st0) + t.st_off;
      c.coef = GP ? 1.0 : a.f_occ[(int64_t)t.fx * a.n_occ + t.fy];
      c.src = t.src;
      c.dt = a.slots[fdp->slot[t.target]].D;
      c.ds = a.slots[fdp->slot[t.src]].D;
      c.ds0 = a.slots[fdp->slot[t.src]].d;
      c.trans = t.trans;
      c.pad_ = 0;
      tc[tid] = c;
    } else if (tid >= 64 && tid - 64 < f_nt) {
      const int tl = tid - 64;
      const SlotInfo sl = a.slots[fdp->slot[tl]];
      SlotLds c;
      c.kt_off = sl.kt_off;
      c.et_off = sl.et_off;
      c.fpq = a.f_occ[(int64_t)sl.p * a.n_occ + sl.p] + a.f_occ[(int64_t)sl.q * a.n_occ + sl.q];
      c.D = sl.D;
      c.ysub = fdp->ysub[tl];
      c.sym = fdp->sym[tl] ? 1 + sl.unsym : 0;
      c.wgt = fdp->wgt[tl];
      c.tb = fdp->tb[tl];
      c.tx = fdp->tx[tl];
      c.te = GP ? fdp->tg[tl] : fdp->te[tl];
      c.gy = !GP ? nullptr : (c.sym == 2 ? Y0 : a.yfin + fdp->yout) + c.ysub;
      c.b0 = c.b1 = 0;
      if (BASE) {
        c.b0 = base_of(a.slots, a.slots[fdp->slot[2]], tl);
      } else if (!GP && a.base && fdp->warm_in) {  // a trimer: slots 3, 4, 5 its pairs
        if (tl >= 3) {
          c.b0 = base_of(a.slots, sl, 2);
        } else {
          c.b0 = base_of(a.slots, a.slots[fdp->slot[tl == 2 ? 4 : 3]], tl == 0 ? 0 : 1);
          c.b1 = base_of(a.slots, a.slots[fdp->slot[tl == 0 ? 4 : 5]], tl == 2 ? 1 : 0);
        }
      }
      sc[tl] = c;
    }
    __syncthreads();
    if (GP) {
      // the pass reads the stored Y in place; the contraction weights 2Y -
      // Y^T = Y~ of the pair targets go to the second scratch buffer, and
      // <Y~_t, Y_t> to gdiag.  A term with a diagonal source p stands for itself,
      // 2 <Y~_t, Z(Y_p)>, and for its mirror, <Y_p + Y_p^T, Z^T(Y_t)> = <Y_t +
      // Y_t^T, Z(Y_p)>: together 4 <Y~_t, Z((3 Y_p + Y_p^T) / 4)>, which differs
      // from 4 <Y~_t, Z(Y_p)> where Y_p is not symmetric; such a source is read
      // from the first scratch buffer
      for (int tl = 0; tl < f_nt; ++tl) {
        const int D = sc[tl].D;
        const int sy = sc[tl].sym;
        const double *y = a.yfin + fdp->yout + sc[tl].ysub;
        double *out = Y0 + (sy ? 0 : ny_cap) + sc[tl].ysub;
        const double ca = sy ? 0.75 : 2.0, cb = sy ? 0.25 : -1.0;
        double part = 0.0;
        for (int e0 = tid; e0 < D * D; e0 += 4 * NTH) {
          double yv[4], yt[4];  // eight loads in flight
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * NTH < D * D ? e0 + u * NTH : e0;
            const int i = e / D, j = e - i * D;
            yv[u] = y[e];
            yt[u] = y[j * D + i];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (e0 + u * NTH < D * D) {
              if (sy != 1) out[e0 + u * NTH] = ca * yv[u] + cb * yt[u];
              part += (2.0 * yv[u] - yt[u]) * yv[u];
            }
        }
        const double tot = wg_sum<NW>(part, red_d);  // also orders these writes
        if (tid == 0) a.gdiag[6 * fi + tl] = tot;
      }
      hasY = true;
    } else if (BASE || (fdp->warm_in && a.warm)) {
      hasY = true;
    }
    // a warm-started fragment's first sweep reads the solutions of its own
    // pairs' fragments in place (warm store, one D x D block per slot)
    bool wsrc = BASE || (!GP && fdp->warm_in && a.warm);
    for (int it = 0;; ++it) {
      double mres = 0.0, epart = 0.0;
      int bad = 0;
      double *const Ycb = Y0 + (cur ? ny_cap : 0);
      double *const Ynb = Y0 + (cur ? 0 : ny_cap);
      // a warm-started trimer's first sweep: the terms within its pairs' own
      // fragments are summed already
      const bool bsrc = !BASE && !GP && wsrc && a.base;
      // the current amplitudes of target / source slot tl
      auto ysrc = [&](int tl) -> const double * {
        if (GP) return sc[tl].gy;
        return wsrc ? a.warm + sc[tl].kt_off : Ycb + sc[tl].ysub;
      };

      // ---- panel pipeline: step (ti, m) = rows 16m.. of S~ and of Y^(T) ----
      // S~ is one contiguous copy, panel after panel; Y's rows likewise, or
      // (transposed source) strips of 16 columns, kept as strips of pitch
      // YPITCH in LDS and read across.  Everything that does not change from
      // panel to panel is set once per term.
      int p_tl = -1, p_ti = 0, p_end = 0, p_m = 0;  // step held in ps, py
      int p_dt = 0, p_ds = 16, p_yv = 0, p_yu = 0, p_ys = 0;
      __amdgpu_buffer_rsrc_t p_rs, p_ry;
      auto open_term = [&]() {  // first term of the next targets that have any
        while (p_ti >= p_end && ++p_tl < f_nt) {
          p_ti = uniform(bsrc ? sc[p_tl].tx : sc[p_tl].tb);
          p_end = uniform(sc[p_tl].te);
        }
        if (p_tl >= f_nt) return;
        const TermLds &tm = tc[p_ti];
        p_dt = uniform(tm.dt);
        p_ds = uniform(tm.ds);
        const bool tr = uniform(tm.trans) != 0;
        p_rs = make_rsrc(uniform(tm.st), p_ds * p_dt * 8);
        p_ry = make_rsrc(uniform(ysrc(tm.src)), p_ds * p_ds * 8);
        p_yv = tr ? (tid >> 3) * p_ds * 8 + (tid & 7) * 16 : tid * 16;
        p_yu = tr ? NTH * p_ds : NTH * 16;
        p_ys = tr ? 128 : 128 * p_ds;
      };
      auto load_panel = [&]() {
        const int so = p_m * 128 * p_dt, yo = p_m * p_ys;
#pragma unroll
        for (int u = 0; u < PFN; ++u) {
          const int e = tid + NTH * u;
          ps[u] = load_b128(p_rs, e < 8 * p_dt ? e * 16 : OOB, so);
        }
#pragma unroll
        for (int u = 0; u < PFN; ++u) {
          const int e = tid + NTH * u;
          py[u] = load_b128(p_ry, e < 8 * p_ds ? p_yv + u * p_yu : OOB, yo);
        }
      };
      if (hasY) {
        open_term();
        if (p_tl < f_nt) load_panel();
      }

      for (int tl = 0; tl < f_nt; ++tl) {
        const SlotLds sl = sc[tl];
        const int Dt = uniform(sl.D);
        const int nT = Dt >> 4;
        const RowPart rp = row_part<NW>(nT, wave);
        const bool row2 = ROW2 && nT == 5;
        d4 acc[SPLIT], acc2[SPLIT];  // MAXNT, NR2 used
#pragma unroll
        for (int jb = 0; jb < MAXNT; ++jb) acc[jb] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int jb = 0; jb < NR2; ++jb) acc2[jb] = d4{0.0, 0.0, 0.0, 0.0};

        if (hasY) {
          const int t_end = uniform(sl.te);
          for (int ti = uniform(bsrc ? sl.tx : sl.tb); ti < t_end;
               ++ti) {
            const double coef = tc[ti].coef;
            const int Ds = uniform(tc[ti].ds);
            const int ds0 = uniform(tc[ti].ds0);
            const bool tr = uniform(tc[ti].trans) != 0;
            const int nS = Ds >> 4;
            // this wave's source blocks: part, part + nparts, ... (cnt of them)
            const int cnt = rp.ib < 0 ? 0 : (nS - rp.part + (1 << rp.lg) - 1) >> rp.lg;
            // the panel's Y part: this thread's place in LDS, its operand reads
            const int yw = tr ? (tid >> 3) * (YPITCH / 2) + (tid & 7) : tid;  // in d2
            const int ywu = tr ? (NTH / 8) * (YPITCH / 2) : NTH;
            const int yk = tr ? 16 * YPITCH : 16, ym = tr ? 4 : 4 * Ds;
            const int yr = (tr ? l16 * YPITCH + lq : lq * Ds + l16) + rp.part * yk;
            const int ystep = yk << rp.lg;
            d4 W[SPLIT], W2[SPLIT];  // MAXNT, NW2 used
#pragma unroll
            for (int kb = 0; kb < MAXNT; ++kb) W[kb] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kb = 0; kb < NW2; ++kb) W2[kb] = d4{0.0, 0.0, 0.0, 0.0};
            __syncthreads();  // the previous term's S~ is no longer read
            for (int mp = 0; mp < nS; ++mp) {
              double *const yb = (mp & 1) ? yb1 : yb0;
              // the panel in ps, py has landed; waiting here explicitly leaves
              // no load outstanding on any path
              __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
              {
                d2 *s_ = reinterpret_cast<d2 *>(Sl + 16 * mp * Dt) + tid;
                d2 *y_ = reinterpret_cast<d2 *>(yb) + yw;
#pragma unroll
                for (int u = 0; u < PFN; ++u) {
                  const int e = tid + NTH * u;
                  if (e < 8 * Dt) s_[NTH * u] = ps[u];
                  if (e < 8 * Ds) y_[ywu * u] = py[u];
                }
              }
              // the next panel streams in under the products; a term's last
              // panel prefetches the next term's first one
              if (++p_m >= (p_ds >> 4)) {
                p_m = 0;
                ++p_ti;
                open_term();
              }
              if (p_tl < f_nt) load_panel();
              __syncthreads();
              if (cnt > 0) {
                const lds_d *sp = as_lds(Sl + (16 * mp + lq) * Dt + l16);
                const lds_d *yp = as_lds(yb + yr);
                double yv = *yp;
                d4 b1, b2 = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int mm = 0; mm < 4; ++mm) {
                  b1[mm] = sp[mm * 4 * Dt + rp.ib * 16];
                  if (ROW2) b2[mm] = sp[mm * 4 * Dt + (row2 ? 64 : 0)];
                }
#pragma unroll
                for (int mm = 0; mm < 4; ++mm) {
                  const double bv = b1[mm], bv2 = b2[mm];
                  const bool on = mm == 0 || 16 * mp + 4 * mm < ds0;  // else zeros
                  const int cm = on ? cnt : 0;
#pragma unroll
                  for (int u = 0; u < MAXNT; ++u) {
                    // the next product's operand is on its way before this one
                    // (past this wave's blocks: its first, unused)
                    const double yn = u + 1 < MAXNT
                                          ? yp[mm * ym + (u + 1 < cnt ? (u + 1) * ystep : 0)]
                                      : mm + 1 < 4  ? yp[(mm + 1) * ym]
                                                    : 0.0;
                    if (__builtin_expect(cm > u, 1)) {
                      W[u] = mfma_f64(yv, bv, W[u]);
                      if (ROW2 && row2 && (u & 3) == wave)
                        W2[u >> 2] = mfma_f64(yv, bv2, W2[u >> 2]);
                    }
                    yv = yn;
                  }
                }
              }
              // one Y buffer: the next panel's store waits for these reads
              if (!DBY) __syncthreads();
            }
#pragma unroll
            for (int u = 0; u < MAXNT; ++u) {
              if (cnt > u) {
                const int kr = 16 * (rp.part + (u << rp.lg));  // the block's first row
                const bool r2 = ROW2 && row2 && (u & 3) == wave;
                const lds_d *brow = as_lds(Sl + (kr + lq) * Dt + l16);
                double sv = *brow;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                  const double av = coef * W[u][v];
                  const double av2 = ROW2 ? coef * W2[u >> 2][v] : 0.0;
                  const int cv = v == 0 || kr + 4 * v < ds0 ? nT : 0;
#pragma unroll
                  for (int jb = 0; jb < MAXNT; ++jb) {
                    // (past the row: the next rows or the Y buffer behind, unused)
                    const double sn = jb + 1 < MAXNT ? brow[v * 4 * Dt + (jb + 1) * 16]
                                      : v + 1 < 4    ? brow[(v + 1) * 4 * Dt]
                                                     : 0.0;
                    if (__builtin_expect(cv > jb, 1)) {
                      acc[jb] = mfma_f64(av, sv, acc[jb]);
                      if (ROW2 && r2) acc2[jb] = mfma_f64(av2, sv, acc2[jb]);
                    }
                    sv = sn;
                  }
                }
              }
            }
            if (GP) {
              // this term's product alone, contracted with Y~ = 2Y - Y^T
              const double *Wy = uniform((const double *)(Y0 + ny_cap + sl.ysub));
              double part = 0.0;
#pragma unroll
              for (int jb = 0; jb < MAXNT; ++jb) {
                if (cnt > 0 && jb < nT) {
                  d4 wy;  // four loads in flight (one by one: a sixth of the pass)
#pragma unroll
                  for (int v = 0; v < 4; ++v)
                    wy[v] = at(Wy, (rp.ib * 16 + lq + 4 * v) * Dt + jb * 16 + l16);
#pragma unroll
                  for (int v = 0; v < 4; ++v) part += wy[v] * acc[jb][v];
                }
                acc[jb] = d4{0.0, 0.0, 0.0, 0.0};
              }
              if (row2) {
#pragma unroll
                for (int jb = 0; jb < NR2; ++jb) {
#pragma unroll
                  for (int v = 0; v < 4; ++v)
                    part += at(Wy, (64 + lq + 4 * v) * Dt + jb * 16 + l16) * acc2[jb][v];
                  acc2[jb] = d4{0.0, 0.0, 0.0, 0.0};
                }
              }
              const double tot = wg_sum<NW>(part, red_d);
              if (tid == 0) a.gterm[f_tb + ti] = tot;
            }
          }
        }
        if (GP) continue;  // no residual in the gradient pass

        // ---- the target's sums: shared row blocks added up (a wave then owns
        // the column blocks jb mod nparts == part of its row block) ----
        const int sym = uniform(sl.sym);
        const uint32_t jm = rp.ib < 0 ? 0u : part_mask(rp.part, rp.lg, nT);
        const uint32_t jm2 = row2 ? part_mask(wave, 2, 5) : 0u;
        const bool summed = hasY && !(bsrc && sym);  // some product was added
        // uniform over the workgroup, unlike nparts
        const bool shared = summed && (row2 || nT < (NW == 8 ? 7 : 3));
        if (shared) {
          __syncthreads();  // S~ of the last term is no longer read
          double *o = Sl + wave * 16 * Dt;
#pragma unroll
          for (int jb = 0; jb < MAXNT; ++jb)
            if (jb < nT && (row2 || rp.lg > 0)) {
#pragma unroll
              for (int v = 0; v < 4; ++v)
                o[(lq + 4 * v) * Dt + jb * 16 + l16] = row2 ? acc2[jb][v] : acc[jb][v];
            }
          __syncthreads();
          const int first = row2 ? 0 : rp.first, stride = row2 ? 1 : rp.stride;
          const int np = row2 ? 4 : 1 << rp.lg;
          if (np > 1) {
            const uint32_t own = row2 ? jm2 : jm;
#pragma unroll
            for (int jb = 0; jb < MAXNT; ++jb)
              if (own & (1u << jb)) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                  double t = 0.0;
                  for (int q = 0; q < np; ++q)
                    t += Sl[((first + stride * q) * 16 + lq + 4 * v) * Dt + jb * 16 + l16];
                  if (row2) acc2[jb][v] = t;
                  else acc[jb][v] = t;
                }
              }
          }
        }
        if (sym && summed) {  // diagonal pair: R~ gets acc + acc^T (mirror terms)
          __syncthreads();  // S~ of the last term, the shares are no longer read
#pragma unroll
          for (int jb = 0; jb < MAXNT; ++jb) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              if (jm & (1u << jb))
                Sl[(rp.ib * 16 + lq + 4 * v) * Dt + jb * 16 + l16] = acc[jb][v];
              if (ROW2 && (jm2 & (1u << jb)))
                Sl[(64 + lq + 4 * v) * Dt + jb * 16 + l16] = acc2[jb][v];
            }
          }
          __syncthreads();
        }

        // ---- residual, energy, update for the owned blocks of target tl ----
        const double *Yc = uniform(ysrc(tl));
        double *Yn = const_cast<double *>(uniform((const double *)(Ynb + sl.ysub)));
        const double *Kt = uniform((const double *)(a.kt + sl.kt_off));
        const double *et = uniform((const double *)(a.et + sl.et_off));
        const double *bs0 = uniform((const double *)(a.base + sl.b0));
        const double *bs1 = uniform((const double *)(a.base + sl.b1));
        const double fpq = uniform(sl.fpq);
        const double w = (double)uniform(sl.wgt);
        // the inputs of block (ib, jb), fetched one block ahead of their use;
        // blocks that are not this wave's fetch one of the target all the same
        struct In {
          d4 k, y, yt, b;
          double ej;
        };
        // no load is under a condition: they all leave together
        const double *const Yq = hasY ? Yc : Kt;  // T = 0: read, not used
        auto fetch = [&](int ib, int jb, auto with_base) {
          In f;
          const int j = jb * 16 + l16, i0 = ib * 16 + lq;
          f.ej = at(et, j);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int ij = (i0 + 4 * v) * Dt + j;
            // Y_pp is symmetric where K~_pp is (its other terms are made so)
            const int ji = sym == 1 ? ij : j * Dt + i0 + 4 * v;
            f.k[v] = at(Kt, ij);
            f.y[v] = at(Yq, ij);
            f.yt[v] = at(Yq, ji);
            if (decltype(with_base)::value) {  // b1 of a pair slot: read, not used
              const double b2 = at(bs1, ij);
              f.b[v] = at(bs0, ij) + (sym ? b2 : 0.0);
            }
          }
          return f;
        };
        auto finish = [&](int ib, int jb, const d4 &t, const In &f, const d4 &ei,
                          auto with_base) {
          const int j = jb * 16 + l16;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int i = ib * 16 + lq + 4 * v;
            double sacc = t[v];
            if (decltype(with_base)::value) sacc += f.b[v];
            else if (sym && summed) sacc += Sl[j * Dt + i];
            const double y = hasY ? f.y[v] : 0.0, yt = hasY ? f.yt[v] : 0.0;
            const double den = fpq - ei[v] - f.ej;
            const double r = f.k[v] - den * y - sacc;
            const double ar = fabs(r);
            if (!(ar <= 1e300)) bad = 1;
            mres = fmax(mres, ar);
            epart += w * (2.0 * y - yt) * (f.k[v] + r);
            put(Yn, i * Dt + j, y + r / den);
          }
        };
        auto finish_row = [&](int ib, uint32_t own, const d4 *t, auto last) {
          constexpr int NB = decltype(last)::value;
          if (BASE) {
            double *o = const_cast<double *>(bs0);
#pragma unroll
            for (int jb = 0; jb < NB; ++jb)
              if (own & (1u << jb)) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                  const int i = ib * 16 + lq + 4 * v, j = jb * 16 + l16;
                  put(o, i * Dt + j, sym ? t[jb][v] + Sl[j * Dt + i] : t[jb][v]);
                }
              }
            return;
          }
          d4 ei;
#pragma unroll
          for (int v = 0; v < 4; ++v) ei[v] = at(et, ib * 16 + lq + 4 * v);
          auto go = [&](auto with_base) {
            In cur = fetch(ib, 0, with_base);
#pragma unroll
            for (int jb = 0; jb < NB; ++jb) {
              In nxt;  // past the last block the first again, unused
              if (jb + 1 < NB) nxt = fetch(ib, jb + 1 < nT ? jb + 1 : 0, with_base);
              if (own & (1u << jb)) finish(ib, jb, t[jb], cur, ei, with_base);
              if (jb + 1 < NB) cur = nxt;
            }
          };
          if (bsrc) go(std::true_type());
          else go(std::false_type());
        };
        if (jm) finish_row(rp.ib, jm, acc, std::integral_constant<int, MAXNT>());
        if (ROW2 && jm2) finish_row(4, jm2, acc2, std::integral_constant<int, NR2>());
      }
      if (GP || BASE) {
        __syncthreads();  // the scratch is read; the next fragment refills it
        break;
      }
      // block reductions (fixed order: deterministic)
      for (int o = 32; o > 0; o >>= 1) {
        mres = fmax(mres, __shfl_xor(mres, o));
        epart += __shfl_xor(epart, o);
        bad |= __shfl_xor(bad, o);
      }
      if (lane == 0) {
        red_d[wave] = mres;
        red_d[NW + wave] = epart;
        red_i[wave] = bad;
      }
      __syncthreads();  // also orders this sweep's Y writes before the next
      const double M = wave_tree_max<NW>(red_d);
      const double E = wave_tree_sum<NW>(red_d + NW);
      int B = 0;
#pragma unroll
      for (int w2 = 0; w2 < NW; ++w2) B |= red_i[w2];
      __syncthreads();
      const bool conv = M < a.tol;
      if (conv || B || it >= a.max_iter) {
        if (tid == 0) {
          a.e_frag[f_frag] = B ? __builtin_nan("") : E;
          a.iters[f_frag] = conv && !B ? it : -(a.max_iter + 1);
          int32_t *st = a.status + 2 * blockIdx.x;  // owned by this workgroup
          if (B) st[0] = 1;
          if (!conv && !B) st[1] = 1;
        }
        if (fdp->warm_out >= 0 && a.warm) {
          // the fragment's own pair seeds the trimers that contain it: its
          // last amplitudes, converged or not (zero after a non-finite
          // residual), so every trimer starts from defined values
          const SlotLds sl = sc[fdp->warm_out];
          const double *src = ysrc(fdp->warm_out);
          for (int e = tid; e < sl.D * sl.D; e += NTH)
            a.warm[sl.kt_off + e] = hasY && !B ? src[e] : 0.0;
        }
        if (ST && conv && !B) {
          // the converged amplitudes (zero if converged at T = 0) for the
          // gradient pass
          for (int tl = 0; tl < f_nt; ++tl) {
            const int D = sc[tl].D;
            const double *src = ysrc(tl);
            double *dst = a.yfin + fdp->yout + sc[tl].ysub;
            for (int e = tid; e < D * D; e += NTH) dst[e] = hasY ? src[e] : 0.0;
          }
        }
        __syncthreads();  // the scratch is read; the next fragment refills it
        break;
      }
      hasY = true;
      wsrc = false;
      cur ^= 1;
    }
  }
}

// Cleared status words, and SlotInfo::unsym: whether K~_pp is unsymmetric (1) or
// symmetric to 2^-36 of its largest element (0): what that leaves of <Y - Y^T, K~>
// is below the rounding of the energy (a NaN ends the fragment anyway).  pair_K's
// blocks are symmetric to rounding, and their transposed Y need not be read: 148.8 ms
// instead of 149.9 for the 160-orbital step, 166.2 instead of 168.7 for 96 orbitals
// of 24 - 64 OSVs.
__global__ __launch_bounds__(1024) void solve_begin_kernel(SlotInfo *__restrict__ slots,
                                                           const double *__restrict__ kt,
                                                           int n_occ,
                                                           int32_t *__restrict__ status,
                                                           int n_status) {
  if ((int)blockIdx.x == n_occ) {
    for (int k = threadIdx.x; k < n_status; k += 1024) status[k] = 0;
    return;
  }
  __shared__ double big[16], dif[16];
  const SlotInfo sl = slots[blockIdx.x];
  const double *K = kt + sl.kt_off;
  double b = 0.0, d = 0.0;
  for (int e = threadIdx.x; e < sl.D * sl.D; e += 1024) {
    const int i = e / sl.D, j = e - i * sl.D;
    const double x = K[e], y = K[j * sl.D + i];
    b = fmax(b, fabs(x));
    d = fmax(d, fabs(x - y));
  }
  for (int o = 32; o > 0; o >>= 1) {
    b = fmax(b, __shfl_xor(b, o));
    d = fmax(d, __shfl_xor(d, o));
  }
  if ((threadIdx.x & 63) == 0) {
    big[threadIdx.x >> 6] = b;
    dif[threadIdx.x >> 6] = d;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 16; ++w) {
      b = fmax(b, big[w]);
      d = fmax(d, dif[w]);
    }
    slots[blockIdx.x].unsym = d <= 0x1p-36 * b ? 0 : 1;
  }
}

hipError_t launch_solve_begin(SlotInfo *slots, const double *kt, int n_occ, int32_t *status,
                              int n_status, hipStream_t s) {
  hipLaunchKernelGGL(solve_begin_kernel, dim3((unsigned)n_occ + 1), dim3(1024), 0, s, slots, kt,
                     n_occ, status, n_status);
  return hipGetLastError();
}

int64_t solve_scratch_doubles(int ny_max, int dmax) {
  return 4LL * ny_max + 2LL * dmax * dmax;
}

// Waves per workgroup of the instance for chunks whose widest pair domain
// has NT 16-row blocks: four up to 80-wide domains (two workgroups share a
// CU), eight from 96 on, where the resident S~ block leaves room for one
// workgroup per CU.  Measured on the 512- and 160-LMO lattices against one
// wave per row block of the widest targets (five to eight waves): balanced
// rows but fewer waves to hide the panel loads, 3% and 20% slower.
template <int NT>
constexpr int solve_waves() { return NT <= 5 ? 4 : 8; }

// LDS of one workgroup: the resident S~ block and two 16-row Y panel
// buffers, one for the 128-wide instance (two would not leave room).
size_t solve_lds_bytes(int dmax) {
  const int ybuf = dmax <= 112 ? 2 * YPITCH : YPITCH;
  // at 16 also the four shares of a target's one row block
  return (size_t)std::max(dmax * dmax + ybuf * dmax, 64 * 16) * sizeof(double);
}

template <int NT, int MODE, int NW>
static hipError_t launch_nt_g(const SolveArgs &a, int n_wg, hipStream_t s, int *per_cu) {
  const size_t smem = solve_lds_bytes(a.dmax);
  hipError_t e = hipFuncSetAttribute((const void *)solve_kernel<NT, MODE, NW>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)smem);
  if (e != hipSuccess) return e;
  if (per_cu)  // resident workgroups per CU for this instance
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(
        per_cu, (const void *)solve_kernel<NT, MODE, NW>, 64 * NW, smem);
  hipLaunchKernelGGL((solve_kernel<NT, MODE, NW>), dim3(n_wg), dim3(64 * NW), smem, s, a);
  return hipGetLastError();
}

template <int MODE>
static hipError_t launch_mode(const SolveArgs &a, int n_wg, hipStream_t s, int *per_cu) {
  if (!per_cu && a.n_frag <= 0) return hipSuccess;
  if (solve_lds_bytes(a.dmax) > 150 * 1024) return hipErrorInvalidValue;
  switch (a.dmax / 16) {
    case 1:
    case 2: return launch_nt_g<2, MODE, solve_waves<2>()>(a, n_wg, s, per_cu);
    case 3: return launch_nt_g<3, MODE, solve_waves<3>()>(a, n_wg, s, per_cu);
    case 4: return launch_nt_g<4, MODE, solve_waves<4>()>(a, n_wg, s, per_cu);
    case 5: return launch_nt_g<5, MODE, solve_waves<5>()>(a, n_wg, s, per_cu);
    case 6: return launch_nt_g<6, MODE, solve_waves<6>()>(a, n_wg, s, per_cu);
    case 7: return launch_nt_g<7, MODE, solve_waves<7>()>(a, n_wg, s, per_cu);
    case 8: return launch_nt_g<8, MODE, solve_waves<8>()>(a, n_wg, s, per_cu);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_solve(const SolveArgs &a, int n_wg, hipStream_t s) {
  return a.yfin ? launch_mode<1>(a, n_wg, s, nullptr) : launch_mode<0>(a, n_wg, s, nullptr);
}

hipError_t launch_solve_base(const SolveArgs &a, int n_wg, hipStream_t s) {
  if (!a.warm || !a.base) return hipErrorInvalidValue;
  return launch_mode<3>(a, n_wg, s, nullptr);
}

hipError_t launch_solve_grad(const SolveArgs &a, int n_wg, hipStream_t s) {
  if (!a.yfin || !a.gterm || !a.gdiag) return hipErrorInvalidValue;
  return launch_mode<2>(a, n_wg, s, nullptr);
}

hipError_t solve_blocks_per_cu(const SolveArgs &a, int mode, int *per_cu) {
  *per_cu = 0;
  switch (mode) {
    case 0: return launch_mode<0>(a, 0, nullptr, per_cu);
    case 1: return launch_mode<1>(a, 0, nullptr, per_cu);
    case 3: return launch_mode<3>(a, 0, nullptr, per_cu);
    default: return launch_mode<2>(a, 0, nullptr, per_cu);
  }
}

}  // namespace mbe3
