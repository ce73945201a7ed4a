// HIP kernels of the graph-PEPS simple update for gfx950 (CDNA4).
//
// One two-qubit gate on edge e = (i, j) is three launches over every
// (instance, edge) work item of a colour class (Method section: simple
// update with the lambda weights as environment, bond dimension chi = D):
//
//   k_absorb_gram per (item, end, physical slice p): absorb the lambda weights
//   / k_absorb_qr of the other legs into Gamma^(p) and reduce the resulting
//                 [M x D_e] matrix A to an R factor with R^H R = A^H A in
//                 float64: Gram matrix on the matrix cores + Cholesky for
//                 complex64 storage, Householder (rows streamed in chunks, R
//                 only) for complex128;
//   k_theta_svd   per item: Theta' = R_i diag(lambda_e) R_j^T times the
//                 diagonal RZZ phase, one-sided Jacobi SVD in float64 held in
//                 LDS, truncation to <= D values with lambda_e <- s/||s||, and
//                 the small re-absorb matrices T (below);
//   k_reabsorb_mfma / k_reabsorb  per (item, end, slice, row block):
//                 Gamma'^(p) = Gamma^(p) T^(p).
//
// Why per-slice QR and T.  RZZ is diagonal in (s, t), so the physical index of
// each end passes through the gate unchanged.  Reducing each physical slice
// A^(p) = Q^(p) R^(p) separately gives block-diagonal isometries, so the
// singular values and vectors of the two-site tensor equal those of the
// smaller Theta'[(a,s),(t,b)] = g(s,t) sum_k R_i^(s)[a,k] lambda_k R_j^(t)[b,k].
// The new tensor of end i, Q_i U with the environment divided out again,
// equals Gamma_i^(s) T_i^(s) with
//   T_i^(s)[k,k'] = lambda_k / sigma_k' * sum_{t,b} g(s,t) R_j^(t)[b,k] V[(t,b),k']
// (and T_j^(t) likewise from conj(U) and R_i), because Q^H A = R.  Q is never
// formed and no division by a neighbouring lambda is needed: the weights
// absorbed into A cancel exactly against the ones the simple update divides out.
//
// Remaining kernels: RX layer (Eq. 2), mean-field <Z> readout (lambda^2 on
// every leg), product-state reset (Eq. 3) and the history step counter.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "gpeps_device.h"
#include "gpeps_internal.h"

namespace gpeps {

hipError_t launch_svd_big(bool c128, const DevState& st, const int32_t* items, int first, int count,
                          hipStream_t stream);

// ------------------------------------------------------------------ K1: absorb + QR

// Workgroup of 256 threads for at most NC columns: lane group c = tid / (256 / NC) owns
// column c of the current row chunk, lane g of the group rows g, g + 256 / NC, ... .  The
// chunk is stacked under the running upper-triangular R (kept in LDS) and reduced column by
// column with complex Householder reflectors P = I - tau v v^H, v = x - beta e_0,
// beta = -phase(x_0) ||x||.  One barrier per column: the group of column j + 1 publishes its
// chunk rows (already updated by reflector j) and their squared norm while the others apply
// reflector j, and every group rebuilds reflector j + 1 from that copy (bit-identical in all
// groups).  A column whose chunk part is exactly zero is skipped, so exact zeros stay exact.
template <typename CT, int NC, int RPT>
__global__ __launch_bounds__(256) void k_absorb_qr(DevState st, const int32_t* __restrict__ items, int first) {
  constexpr int LPC = 256 / NC;  // lanes per column (RPT: rows per lane per chunk)
  constexpr int CH = LPC * RPT;  // rows per chunk
  int slot, side, p;
  end_task(st, blockIdx.x, slot, side, p);
  const int e = items[first + slot];
  const EdgeInfo& E = st.edges[e];
  const SideGeom G = side_geom(st, E.side[side]);
  const int n = st.chi[e];
  const int M = G.d1 * G.d2;
  const CT* gam = reinterpret_cast<const CT*>(st.gamma);
  double2* R = st.rbuf + rbuf_off(st, slot, side, p);
  const int D = st.D;
  const int tid = threadIdx.x;

  if (M <= n) {  // no reduction: R = A (M x n)
    for (int idx = tid; idx < M * n; idx += blockDim.x) {
      const int m = idx / n, k = idx - (idx / n) * n;
      R[m * D + k] = cscale(to_d2(gam[G.addr(p, m, k)]), G.env(m));
    }
    return;
  }

  __shared__ double2 Rm[NC][NC + 1];
  __shared__ double2 vb[2][CH];  // chunk rows of the next pivot column, by step parity
  __shared__ double vn[2];        // and their squared norm

  const int c = tid / LPC;
  const int g = tid - (tid / LPC) * LPC;
  for (int idx = tid; idx < NC * (NC + 1); idx += blockDim.x) (&Rm[0][0])[idx] = make_double2(0.0, 0.0);

  double2 x[RPT];
  for (int r0 = 0; r0 < M; r0 += CH) {
    // every load of the chunk is issued before the first use: addresses are clamped into the
    // matrix and rows or columns outside it are zeroed afterwards
    const int cc = c < n ? c : n - 1;
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
      const int m = r0 + g + LPC * i;
      const int mc = m < M ? m : M - 1;
      const double2 a = cscale(to_d2(gam[G.addr(p, mc, cc)]), G.env(mc));
      x[i] = (c < n && m < M) ? a : make_double2(0.0, 0.0);
    }
    if (c == 0) {
      double sp = 0.0;
#pragma unroll
      for (int i = 0; i < RPT; ++i) {
        vb[0][g + LPC * i] = x[i];
        sp += cabs2(x[i]);
      }
      sp = group_sum_dpp(sp, LPC);
      if (g == 0) vn[0] = sp;
    }
    bool set_diag = false;  // this group's column got a new diagonal in this chunk
    double2 my_beta = make_double2(0.0, 0.0);
    __syncthreads();
    for (int j = 0; j < n; ++j) {
      const double2* vj = vb[j & 1];
      const double2 alpha = Rm[j][j];
      double2 v[RPT];
#pragma unroll
      for (int i = 0; i < RPT; ++i) v[i] = vj[g + LPC * i];
      const double s2 = vn[j & 1];  // squared norm of the pivot column's chunk part
      if (s2 > 0.0) {
        const double aa2 = cabs2(alpha);
        const double nu2 = aa2 + s2;
        const double nu = nu2 * rsq_nr(nu2);
        const double2 ph = aa2 > 0.0 ? cscale(alpha, rsq_nr(aa2)) : make_double2(1.0, 0.0);
        const double2 beta = cscale(ph, -nu);
        const double2 v0 = csub(alpha, beta);
        const double tau = 2.0 * rcp_nr(cabs2(v0) + s2);
        if (c == j) {
          set_diag = true;
          my_beta = beta;
        } else if (c > j && c < n) {
          double wr = 0.0, wi = 0.0;
#pragma unroll
          for (int i = 0; i < RPT; ++i) {
            const double2 t = cmulc(v[i], x[i]);
            wr += t.x;
            wi += t.y;
          }
          double2 rjc = make_double2(0.0, 0.0);
          if (g == 0) {
            rjc = Rm[j][c];
            const double2 t = cmulc(v0, rjc);
            wr += t.x;
            wi += t.y;
          }
          group_sum2_dpp(wr, wi, LPC);
          const double2 f = make_double2(wr * tau, wi * tau);
#pragma unroll
          for (int i = 0; i < RPT; ++i) x[i] = csub(x[i], cmul(v[i], f));
          if (g == 0) Rm[j][c] = csub(rjc, cmul(v0, f));
        }
      }
      if (c == j + 1) {
        double sp = 0.0;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
          vb[(j + 1) & 1][g + LPC * i] = x[i];
          sp += cabs2(x[i]);
        }
        sp = group_sum_dpp(sp, LPC);
        if (g == 0) vn[(j + 1) & 1] = sp;
      }
      __syncthreads();
    }
    if (set_diag && g == 0) Rm[c][c] = my_beta;
  }
  __syncthreads();
  for (int idx = tid; idx < n * n; idx += blockDim.x) {
    const int a = idx / n, k = idx - (idx / n) * n;
    R[a * D + k] = (k >= a) ? Rm[a][k] : make_double2(0.0, 0.0);
  }
}

// ------------------------------------------------------------------ K1 (complex64): absorb + Gram / Cholesky

// Complex64 storage takes R from the Gram matrix: G = A^H A (A = Gamma^(p) with the other legs'
// lambdas on its rows) on the FP64 matrix cores, then R^H R = G by Cholesky.  Only R^H R enters
// the update (the spectrum of Theta' and the new tensors are unchanged by R -> W R, W unitary),
// so this R serves as the Householder one does.  With v_mfma_f64_16x16x4f64 lane l holds
// A[l % 16][l / 16] and B[l / 16][l % 16] and receives D[l / 16 + 4 r][l % 16]; the reduction
// index (the row m of A) is l / 16, so a lane holds A[m][k] for one column k of each 16-column
// tile and the same registers serve both operands.  Each wave sums a quarter of the rows; the
// four partial Gram matrices are added in LDS in a fixed order.  G rounds at ~2^-53 ||A||^2:
// directions of A below ~1e-7 of its norm are not resolved, about the complex64 rounding of the
// stored tensors, and a Cholesky pivot below 1e-13 of its column's squared norm is taken as
// zero (that row of R is zero), which keeps exact zeros exact.
//
// Above D = 32 the rows of an end go to kGramSplit workgroups where the whole context has few edges
// (st.gram_split): an end with three legs has up to 4096 rows, the few such ends of a class leave most
// CUs idle, and one CU's FP64 matrix cores need 250 us for one.  The first launch (kGramPart) leaves
// the partial Gram matrices in the scratch of the SVD that follows, the second (kGramEnd) adds them in a
// fixed order and factorises.  One 127-qubit instance at D = 64: 479 -> 217 + 85 us in the largest
// class, 147 -> 104 us in the mean.  Ends of at most kGramSplitRows rows are done whole by the first
// launch, and only the tiles that the bond fills are written: while the bonds are small the partial
// sums cost more than the rows.  One 127-qubit instance at D = 33, microseconds of the first eight steps:
// 27 / 32 / 34 / 38 / 59 / 94 / 96 / 96 with every end split and every tile written,
// 14 / 19 / 26 / 34 / 58 / 94 / 97 / 98 from 8 rows, 14 / 16 / 19 / 29 / 56 / 92 / 97 / 97 from 128,
// 14 / 16 / 19 / 31 / 63 / 92 / 97 / 97 from 512.
constexpr int kGramWhole = 0, kGramPart = 1, kGramEnd = 2;
constexpr int kGramSplit = 4;
constexpr int kGramSplitRows = 128;

template <int NC, int MODE = kGramWhole>
__global__ __launch_bounds__(256, NC == 32 ? 4 : 1) void k_absorb_gram(DevState st, const int32_t* __restrict__ items, int first) {
  typedef double d4 __attribute__((ext_vector_type(4)));
  constexpr int NT16 = NC / 16;                 // column tiles of 16
  constexpr int NTILE = NT16 * (NT16 + 1) / 2;  // tiles on and above the diagonal
  constexpr int UNR = NT16 >= 4 ? 2 : 4 / NT16;  // row steps (of 4 rows) per load batch in flight
  int slot, side, p;
  constexpr int SP = MODE == kGramPart ? kGramSplit : 1;
  // the parts of an end lie a whole grid of ends apart: the ends done whole then stand in consecutive
  // blocks, on all XCDs (block mod 8)
  const int ends = (int)gridDim.x / SP;
  const int split = MODE == kGramPart ? (int)blockIdx.x / ends : 0;
  end_task(st, blockIdx.x - split * ends, slot, side, p);
  const int e = items[first + slot];
  const EdgeInfo& E = st.edges[e];
  const SideGeom G = side_geom(st, E.side[side]);
  const int n = st.chi[e];
  const int M = G.d1 * G.d2;
  const float2* gam = reinterpret_cast<const float2*>(st.gamma);
  double2* R = st.rbuf + rbuf_off(st, slot, side, p);
  const int D = st.D;
  const int tid = threadIdx.x;

  const bool whole = MODE == kGramWhole || M <= kGramSplitRows;
  if ((MODE == kGramPart && whole && split > 0) || (MODE == kGramEnd && whole)) return;
  if (M <= n) {  // no reduction: R = A (M x n)
    for (int idx = tid; idx < M * n; idx += 256) {
      const int m = idx / n, k = idx - (idx / n) * n;
      R[m * D + k] = cscale(to_d2(gam[G.addr(p, m, k)]), G.env(m));
    }
    return;
  }

  // LDS: the partial tiles of waves 2 and 3 (part0 | part1), then the upper triangle of G,
  // which overlaps part1 only: part1 is dead once wave 1 has added it, and wave 0 reads part0
  // while it writes G.
  constexpr int PART = NTILE * 4 * 64;
  constexpr int GSZ = NC * (NC + 1);
  static_assert(MODE == kGramWhole || 4 * kGramSplit * PART <= big_scratch(NC), "partial sums in st.big");
  __shared__ double2 lds[PART + (GSZ > PART ? GSZ : PART)];
  __shared__ double dg[NC];           // squared column norms (diagonal of G)
  __shared__ double envs[2][NC];      // lambda weights of the other two legs (1 for a missing leg)
  double2* part0 = lds;
  double2* part1 = lds + PART;
  auto Gs = [&](int i, int j) -> double2& { return lds[PART + i * (NC + 1) + j]; };

  double2* const gpar = MODE == kGramWhole ? nullptr
                                           : st.big + (int64_t)slot * big_scratch(D) + (side * 2 + p) * kGramSplit * PART;
  if (tid < NC) {
    envs[0][tid] = (G.l1 && tid < G.d1) ? G.l1[tid] : 1.0;
    envs[1][tid] = (G.l2 && tid < G.d2) ? G.l2[tid] : 1.0;
  }
  __syncthreads();

  const int l = tid & 63, wv = tid >> 6, li = l & 15, lk = l >> 4;
  if constexpr (MODE != kGramEnd) {
  d4 gr[NTILE], gi[NTILE];
#pragma unroll
  for (int t = 0; t < NTILE; ++t) {
    gr[t] = (d4){0.0, 0.0, 0.0, 0.0};
    gi[t] = (d4){0.0, 0.0, 0.0, 0.0};
  }
  const int WS = whole ? 4 : 4 * SP;  // waves that share the rows
  // Software pipelined: the complex64 elements of the next batch of rows (4 ks + l / 16, columns
  // 16 t + l % 16) are in flight while the products of the current batch run.  A row past the
  // end gets weight 0 (its load is clamped to the last row).
  const int ksteps = (M + 3) >> 2;
  const int64_t pbase = G.base + p * G.pstride;
  float2 nx[UNR][NT16];
  double nw[UNR];
  auto fetch = [&](int ks0) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int m = 4 * (ks0 + WS * u) + lk;
      const bool mv = m < M;
      const int mc = mv ? m : M - 1;
      const int o1 = mc / G.d2, o2 = mc - (mc / G.d2) * G.d2;
      nw[u] = mv ? envs[0][o1] * envs[1][o2] : 0.0;
      const int64_t ro = pbase + (int64_t)o1 * G.s1 + (int64_t)o2 * G.s2;
#pragma unroll
      for (int t = 0; t < NT16; ++t) {
        const int k = 16 * t + li;
        const int kc = k < n ? k : n - 1;
        nx[u][t] = gam[ro + (int64_t)kc * G.sq];
      }
    }
  };
  const int w0 = split * 4 + wv;
  fetch(w0);
  for (int ks0 = w0; ks0 < ksteps; ks0 += WS * UNR) {
    float2 x[UNR][NT16];
    double w[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      w[u] = nw[u];
#pragma unroll
      for (int t = 0; t < NT16; ++t) x[u][t] = nx[u][t];
    }
    if (ks0 + WS * UNR < ksteps) fetch(ks0 + WS * UNR);
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      double2 a[NT16];
#pragma unroll
      for (int t = 0; t < NT16; ++t) {
        const double wt = 16 * t + li < n ? w[u] : 0.0;
        a[t] = make_double2(wt * (double)x[u][t].x, wt * (double)x[u][t].y);
      }
      int tile = 0;
#pragma unroll
      for (int ta = 0; ta < NT16; ++ta)
#pragma unroll
        for (int tb = ta; tb < NT16; ++tb) {
          // G[k][k'] = sum_m conj(A[m][k]) A[m][k']: Re = Ar^T Ar + Ai^T Ai, Im = Ar^T Ai - Ai^T Ar.
          // On a diagonal tile the second term of Im is the transpose of the first, so only
          // X = Ar^T Ai is accumulated there and Im = X - X^T is formed once, after the sum.
          gr[tile] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ta].x, a[tb].x, gr[tile], 0, 0, 0);
          gr[tile] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ta].y, a[tb].y, gr[tile], 0, 0, 0);
          gi[tile] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[ta].x, a[tb].y, gi[tile], 0, 0, 0);
          if (ta != tb) gi[tile] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[ta].y, a[tb].x, gi[tile], 0, 0, 0);
          ++tile;
        }
    }
  }
  // partial sums of the four waves, added in a fixed order: (0 + 2) + (1 + 3)
  if (wv >= 2) {
    double2* part = wv == 2 ? part0 : part1;
#pragma unroll
    for (int t = 0; t < NTILE; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) part[(t * 4 + r) * 64 + l] = make_double2(gr[t][r], gi[t][r]);
  }
  __syncthreads();
  if (wv < 2) {
    const double2* part = wv == 0 ? part0 : part1;
#pragma unroll
    for (int t = 0; t < NTILE; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double2 q = part[(t * 4 + r) * 64 + l];
        gr[t][r] += q.x;
        gi[t][r] += q.y;
      }
  }
  __syncthreads();
  if (wv == 1) {
#pragma unroll
    for (int t = 0; t < NTILE; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) part0[(t * 4 + r) * 64 + l] = make_double2(gr[t][r], gi[t][r]);
  }
  __syncthreads();
  if (wv == 0) {
    int tile = 0;
#pragma unroll
    for (int ta = 0; ta < NT16; ++ta)
#pragma unroll
      for (int tb = ta; tb < NT16; ++tb) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double2 q = part0[(tile * 4 + r) * 64 + l];
          const double2 v = make_double2(gr[tile][r] + q.x, gi[tile][r] + q.y);
          // off the diagonal tiles k < k' always; a diagonal tile is stored whole (its lower
          // half holds X[k'][k] for the antisymmetrisation below)
          if (MODE == kGramPart && !whole) {
            if (16 * tb < n) gpar[split * PART + (tile * 4 + r) * 64 + l] = v;
          } else {
            Gs(16 * ta + lk + 4 * r, 16 * tb + li) = v;
          }
        }
        ++tile;
      }
  }
  } else {
    int tile = 0;
#pragma unroll
    for (int ta = 0; ta < NT16; ++ta)
#pragma unroll
      for (int tb = ta; tb < NT16; ++tb) {
        if ((tile & 3) == wv && 16 * tb < n) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            double2 v = gpar[(tile * 4 + r) * 64 + l];
#pragma unroll
            for (int q = 1; q < kGramSplit; ++q) v = cadd(v, gpar[q * PART + (tile * 4 + r) * 64 + l]);
            Gs(16 * ta + lk + 4 * r, 16 * tb + li) = v;
          }
        }
        ++tile;
      }
  }
  if (MODE == kGramPart && !whole) return;
  __syncthreads();
  // Im G on the diagonal tiles: X[k][k'] - X[k'][k] on the upper triangle (which is all the
  // factorisation reads), exactly 0 on the diagonal; only the upper entries are written
  for (int idx = tid; idx < NT16 * 256; idx += blockDim.x) {
    const int t16 = 16 * (idx >> 8), k = t16 + ((idx >> 4) & 15), kp = t16 + (idx & 15);
    if (k < kp) Gs(k, kp).y -= Gs(kp, k).y;
    else if (k == kp) Gs(k, k).y = 0.0;
  }
  if (tid < n) dg[tid] = Gs(tid, tid).x;
  __syncthreads();
  if constexpr (NC == 16) {
    // One wave, no barriers: lane l holds column j = l % 16 of the upper triangle, rows
    // i = l / 16 + 4 r (r = 0..3); the pivot comes by readlane and row k of R through LDS
    // (same wave, so the write precedes the reads).  The arithmetic is that of the loop below.
    __shared__ double2 rowk[2][16];
    if (wv != 0) return;
    const int j = l & 15, rq = l >> 4;
    double2 gq[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = rq + 4 * r;
      const double2 t = Gs(i, j);
      gq[r] = (i <= j && j < n) ? t : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      if (k < n) {
        const double d = readlane_d(gq[k >> 2].x, k + 16 * (k & 3));  // G[k][k]
        const bool keep = d > 1e-13 * dg[k];
        const double rk = keep ? rsq_nr(d) : 0.0;  // 1 / R[k][k]
        if (rq == (k & 3) && j >= k) {
          const double2 v = j == k ? make_double2(keep ? d * rk : 0.0, 0.0) : cscale(gq[k >> 2], rk);
          gq[k >> 2] = v;
          rowk[k & 1][j] = v;
        }
        wave_lds_sync();  // other lanes read what these lanes wrote
        const double2 rkj = rowk[k & 1][j];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = rq + 4 * r;
          const double2 rki = rowk[k & 1][i];
          if (i > k && i <= j && j < n) gq[r] = csub(gq[r], cmulc(rki, rkj));
        }
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = rq + 4 * r;
      if (i < n && j < n) R[i * D + j] = j >= i ? gq[r] : make_double2(0.0, 0.0);
    }
    return;
  }
  // right-looking Cholesky, R^H R = G, R upper triangular, in place in the upper triangle
  for (int k = 0; k < n; ++k) {
    const double d = Gs(k, k).x;
    const bool keep = d > 1e-13 * dg[k];
    const double rk = keep ? rsq_nr(d) : 0.0;  // 1 / R[k][k]
    __syncthreads();
    if (tid >= k && tid < n) Gs(k, tid) = tid == k ? make_double2(keep ? d * rk : 0.0, 0.0) : cscale(Gs(k, tid), rk);
    __syncthreads();
    const int w = n - k - 1;
    for (int idx = tid; idx < w * w; idx += blockDim.x) {
      const int i = k + 1 + idx / w, j = k + 1 + idx - (idx / w) * w;
      if (i <= j) Gs(i, j) = csub(Gs(i, j), cmulc(Gs(k, i), Gs(k, j)));
    }
    __syncthreads();
  }
  for (int idx = tid; idx < n * n; idx += blockDim.x) {
    const int a = idx / n, k = idx - (idx / n) * n;
    R[a * D + k] = (k >= a) ? Gs(a, k) : make_double2(0.0, 0.0);
  }
}

// ------------------------------------------------------------------ K2: Theta + Jacobi SVD + truncation

// One workgroup of NT = 256 threads per item; NMAX = 2 * largest D handled
// (32 for D <= 16, 64 for D <= 32).  Theta' lives in LDS as the matrix B, the one of Theta' and
// Theta'^H with fewer columns.  B P = Q R with the columns in an order P of falling size, and the
// one-sided (Hestenes) Jacobi iteration runs on X = R^H, whose columns start nearly orthogonal and
// graded: its orthogonalised columns are B's right singular vectors with rows permuted by P, scaled
// by the singular values.  Squared column norms are tracked and recomputed at the start of every
// sweep, so each rotation needs a single reduction (the inner product).  A pair is rotated when its
// inner product exceeds 2^-52 * nB relative to the column norms and also exceeds
// 2^-52 * eps^2 * ||B||_F^2 (eps = truncation cutoff): pairs below that are
// made of columns far under the cutoff (rounding noise), whose rotation
// cannot move a kept singular vector.  The sweep loop ends when a sweep
// applies no rotation, or when every rotation of the sweep was quiet.
//   complex64 (ACC = false): quiet at |g|^2 <= 1e-8 al be (what is left, 1e-8 between separated
// values, is under the 2^-24 rounding of the complex64 tensors the update writes), one Newton step, not
// two, for the reciprocal square roots (unitarity to ~1e-13 per rotation), R from a column-pivoted
// Cholesky factorisation of B^H B, and the other set of singular vectors from the original Theta'
// as U = Theta' V / sigma or V = Theta'^H U / sigma, accurate to ~2^-52 sigma_0 / sigma_k, well
// below the complex64 storage rounding for every kept value (cutoff ~1e-6).
//   complex128 (ACC = true, cutoffs down to 1e-12): quiet at |g|^2 <= 1e-16 al be and
// tan^2 theta <= 1e-16: a later rotation of the sweep then puts at most the product of two such values
// back into a pair already done, so what is left is under the rotation threshold.  The angle has to be
// tested too: values closer to one another than |g| turn by large angles however small g is, and three
// or more of them hand the couplings on undiminished (eight values 1e-9 apart: vectors orthogonal to
// 1.4e-10 without the test of the angle, to 3.5e-15 with it, as after a sweep without rotations; the sweeps of
// separated values are the same).  R from a
// Householder QR of B with its columns sorted by norm, and the rotations accumulated in W, so that
// the other set is Q W, accurate for every sigma.  D = 16, ten steps of the 127-qubit graph: 106 us
// per launch and 5.3 sweeps (9.3 at most 17 without the QR, through LDS: 192 us).  A square B of at
// most kSmallB columns takes Q = I, R = B: there the QR and the reflectors cost more than the sweep
// they save (with 10 columns, D = 5, a launch is 54.6 us with the QR and 57.1 without, with 16 they are even).
// BWD: the forward update (the same path and arithmetic, so the truncation rank and the
// gauge of the new tensors are the forward ones bit for bit) that also keeps what the
// reverse sweep needs: every singular triplet (bU, bV, bS) and float64 T matrices (t64).
constexpr double kJacobiQuietC64 = 1e-8;    // (1e-4)^2: relative size of a quiet rotation, complex64
constexpr int kSmallB = 8;                  // largest square B that skips the QR, complex128
constexpr double kJacobiQuietC128 = 1e-16;  // (1e-8)^2: the same for the complex128 path, and of its tan^2 theta

template <typename CT, int NT, int NMAX, bool ACC_, bool BWD = false>
__global__ __launch_bounds__(NT, NMAX == 64 ? (ACC_ ? 1 : 2) : NT == 256 ? 4 : ACC_ ? 1 : 2) void k_theta_svd(DevState st, const int32_t* __restrict__ items, int first) {
  constexpr bool ACC = ACC_;
  constexpr int DM = NMAX / 2;             // largest bond dimension handled
  constexpr int EPT = NMAX * NMAX / NT;    // Theta' entries per thread (16)
  constexpr int RPT = NMAX * DM / NT;      // singular-vector entries per thread (8)
  constexpr int RPL = NMAX * NMAX / (2 * NT);  // rows per lane of a Jacobi column pair (upper bound)
  static_assert(2 * NT / NMAX <= 64 && RPL * (2 * NT / NMAX) >= NMAX, "Jacobi rows must fit RPL per lane");
  constexpr int DS = DM + 1;               // padded row stride of the staging arena (no bank conflicts)
  // B: column-major B[col][row].  A 16-lane LDS cycle covers all 64 banks once when it reads 16
  // consecutive rows of a column (the Jacobi lane groups at NMAX = 32); the stride at NMAX = 64
  // makes two rows of 8 consecutive columns conflict-free too (the lane groups there), and leaves
  // the Gram products (one row of 16 columns) two-way conflicts instead of 16-way ones: the
  // preconditioning phase 185 -> 160 k cycles.  (An odd stride at NMAX = 32 cost one instance 0.5 us
  // a launch and 128 of them 1 %.)  The same memory is the staging arena of 4 DM DS elements.
  constexpr int BST = NMAX == 32 ? NMAX : NMAX + 2;
  constexpr int kBsz = NMAX * BST > 4 * DM * DS ? NMAX * BST : 4 * DM * DS;
  __shared__ double2 Bmem[kBsz];
  __shared__ double2 Wmem[ACC ? kBsz : 1];  // accumulated rotations W[col][row] (ACC only), also an arena
  double2 (*const B)[BST] = reinterpret_cast<double2 (*)[BST]>(Bmem);
  double2 (*const W)[BST] = reinterpret_cast<double2 (*)[BST]>(Wmem);
  __shared__ double nrm[NMAX];
  __shared__ double scl[NMAX];  // squared scale of a column of B (and W) during the Jacobi sweeps
  __shared__ double lam_old[kMaxD];
  __shared__ double sig[NMAX];
  __shared__ int perm[NMAX];
  __shared__ int sh_chi;
  __shared__ double sh_norm;
  __shared__ double sh_floor;
  __shared__ int colid[NMAX];   // original column of each pivoted position
  __shared__ double red_w[NT / 64];      // per-wave partial sums
  double2* const arena = Bmem;
  double2* const A0 = arena;            // [2 DM DS]
  double2* const A1 = arena + 2 * DM * DS;  // [2 DM DS]

  const int slot = blockIdx.x;
  const int e = items[first + slot];
  const EdgeInfo& E = st.edges[e];
  const InstParam ip = st.inst[E.inst];
  const int D = st.D;
  const int de = st.chi[e];
  double* lam_e = st.lam + (int64_t)e * D;

  int r[2];
  for (int sd = 0; sd < 2; ++sd) {
    const SideInfo& S = E.side[sd];
    const int d1 = S.oth[0] >= 0 ? st.chi[S.oth[0]] : 1;
    const int d2 = S.oth[1] >= 0 ? st.chi[S.oth[1]] : 1;
    r[sd] = min(d1 * d2, de);
  }
  const int ri = r[0], rj = r[1];
  const int m0 = 2 * ri, n0 = 2 * rj;
  const bool trans = n0 > m0;  // orthogonalise the shorter side
  const int mB = trans ? n0 : m0;
  const int nB = trans ? m0 : n0;
  // complex128: 9 to 16 columns keep two waves of the four busy.  Workgroups that share a CU have numbers
  // a multiple of 256 (the CUs) apart and their first waves sit on successive SIMDs, so the second one's
  // busy pair would overlap the first one's: it numbers its waves from the SIMD after.  127 qubits x 8
  // at D = 5 70 -> 63 us, at D = 8 82 -> 71.  (One busy wave is placed best without.)
  const int turn = ACC && NT == 256 && nB > 8 ? (0 - (int)(blockIdx.x >> 8)) & 3 : 0;
  const int tid = (threadIdx.x + 64 * turn) & (NT - 1);
  const bool small_sq = ACC && nB <= kSmallB && mB == nB;
  const double2* Rg = st.rbuf + rbuf_off(st, slot, 0, 0);  // 4 consecutive [D][D] blocks: i0, i1, j0, j1

  // stage the R factors of one end ([2][r][de], row stride DS) into an LDS region
  auto stage_r = [&](double2* dst, int side, int rows) {
    if (NMAX == 64 && 2 * rows * de <= NT) {  // the first steps: one entry a thread
      const int sl = tid / (rows * de), rem = tid - sl * rows * de, rr = rem / de, k = rem - rr * de;
      if (sl < 2) dst[sl * DM * DS + rr * DS + k] = Rg[(side * 2 + sl) * D * D + rr * D + k];
      return;
    }
    constexpr int PT = 2 * DM * DM / NT;  // entries a thread, all in flight
    double2 v[PT];
#pragma unroll
    for (int q = 0; q < PT; ++q) {
      const int idx = tid + q * NT;
      const int sl = idx / (DM * DM), rr = (idx / DM) % DM, k = idx % DM;
      v[q] = Rg[(side * 2 + sl) * D * D + min(rr, rows - 1) * D + min(k, de - 1)];
    }
#pragma unroll
    for (int q = 0; q < PT; ++q) {
      const int idx = tid + q * NT;
      const int sl = idx / (DM * DM), rr = (idx / DM) % DM, k = idx % DM;
      if (rr < rows && k < de) dst[sl * DM * DS + rr * DS + k] = v[q];
    }
  };

  if (tid < kMaxD) lam_old[tid] = tid < de ? lam_e[tid] : 0.0;

  // Theta'[(s,a)][(t,b)] = g(s,t) sum_k R_i^(s)[a,k] lambda_k R_j^(t)[b,k]: the complex product
  // [2 r_i x D_e] [D_e x 2 r_j] on v_mfma_f64_16x16x4f64, four real products per complex one,
  // operands straight from the R factors in global memory.  With that instruction lane l holds
  // A[l % 16][l / 16] and B[l / 16][l % 16] and receives D[l / 16 + 4 r][l % 16], r = 0..3.
  // Each wave takes 16 x 16 output tiles; ||Theta'||_F^2 is reduced on the way.
  {
    typedef double d4 __attribute__((ext_vector_type(4)));
    constexpr int KS = DM / 4;  // k steps of 4 at the largest bond
    const int l = tid & 63, wv = tid >> 6, li = l & 15, lk = l >> 4;
    const int tiles_c = (n0 + 15) >> 4;
    const int ntiles = ((m0 + 15) >> 4) * tiles_c;
    const int ksteps = (de + 3) >> 2;
    double fro = 0.0;
    for (int tile = wv; tile < ntiles; tile += NT / 64) {
      const int tr = tile / tiles_c, tc = tile - (tile / tiles_c) * tiles_c;
      const int rho = 16 * tr + li, kap = 16 * tc + li;
      const bool rv = rho < m0, cv = kap < n0;
      const int s = rv ? rho / ri : 0, a = rv ? rho - s * ri : 0;
      const int t = cv ? kap / rj : 0, b = cv ? kap - t * rj : 0;
      const double2* Ra = Rg + (int64_t)s * D * D + a * D;
      const double2* Rb = Rg + (int64_t)(2 + t) * D * D + b * D;
      double2 x[KS], y[KS];
      double w[KS];
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {  // valid entries only: the loads do not wait for one another
        x[kk] = y[kk] = make_double2(0.0, 0.0);
        w[kk] = 0.0;
        if (NMAX == 32 || kk < ksteps) {  // (uniform)
          const int k = min(4 * kk + lk, de - 1);
          x[kk] = Ra[k];
          y[kk] = Rb[k];
          w[kk] = lam_e[k];
        }
      }
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {
        const int k = 4 * kk + lk;
        x[kk] = (rv && k < de) ? cscale(x[kk], w[kk]) : make_double2(0.0, 0.0);
        y[kk] = (cv && k < de) ? y[kk] : make_double2(0.0, 0.0);
      }
      // The registers x, y serve C = X Y (A = X, B = Y) and C^T = Y^T X^T (A = Y^T, B = X^T)
      // alike; the orientation is chosen so that the 16 lanes sharing an output register
      // store 16 consecutive rows of one column of B.
      d4 cr = {0.0, 0.0, 0.0, 0.0}, ci = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) {
        if (kk < ksteps) {
          // trans: A = X, B = Y (lanes l % 16 <-> kap); else A = Y^T, B = X^T (lanes <-> rho)
          const double2 a = trans ? x[kk] : y[kk];
          const double2 b = trans ? y[kk] : x[kk];
          cr = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, cr, 0, 0, 0);
          cr = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, cr, 0, 0, 0);
          ci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, ci, 0, 0, 0);
          ci = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, ci, 0, 0, 0);
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int ro = trans ? 16 * tr + lk + 4 * r : rho;  // row of Theta'
        const int co = trans ? kap : 16 * tc + lk + 4 * r;  // column of Theta'
        if (ro < m0 && co < n0) {
          const double2 v = cmul(make_double2(cr[r], ci[r]), gate_phase(ip, ro / ri, co / rj));
          fro += cabs2(v);
          if (!trans) B[co][ro] = v;
          else B[ro][co] = cconj(v);
          // the reverse sweep recovers the other vector set through Theta' (kept row-major)
          if (BWD && !ACC) st.wsb[(int64_t)slot * adj_scratch(D) + (int64_t)32 * D * D + ro * 2 * D + co] = v;
        }
      }
    }
    fro = group_sum_dpp(fro, 64);
    if (l == 0) red_w[wv] = fro;
  }
  if (ACC) {
    for (int idx = tid; idx < nB * nB; idx += NT) {
      const int cc = idx / nB, rr = idx - (idx / nB) * nB;
      W[cc][rr] = make_double2(cc == rr ? 1.0 : 0.0, 0.0);
    }
  }
  __syncthreads();
  if (tid == 0) {
    double f = 0.0;
    for (int w = 0; w < NT / 64; ++w) f += red_w[w];
    sh_floor = f * st.trunc_rel * st.trunc_rel * 2.220446049250313e-16;
  }

  // Preconditioning, complex64 path: R from a column-pivoted Cholesky factorisation of the
  // Gram matrix, P^T B^H B P = R^H R, then the Jacobi iteration runs on X = R^H (nB x nB).  With
  // Q = B P R^-1 (orthonormal columns), B P = Q R and X = U_X S W^H gives B = (Q W) S (P U_X)^H,
  // so the orthogonalised columns of X are B's right singular vectors (rows permuted by P) and
  // Q is never needed.  Only R^H R enters, as for the R factors of the absorb kernel: directions
  // of B below ~1e-8 of its norm are not resolved, two orders under the truncation cutoff and
  // about the complex64 rounding of the stored tensors; the factorisation stops at a pivot below
  // 64 eps of the first (the remaining rows of R are zero).
  if constexpr (!ACC) {
    // G = B^H B on the FP64 matrix cores, 16 x 16 tiles over the waves (tile wv + q NW of the
    // tg x tg grid to wave wv; lane l holds rows i0 + l / 16 + 4 r, column j0 + l % 16 of each).
    constexpr int NW = NT / 64;
    constexpr int TPW = ((NMAX / 16) * (NMAX / 16) + NW - 1) / NW;  // tiles per wave (at most)
    const int wv = tid >> 6, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int tg = (nB + 15) >> 4;
    cgemm_d4 sr[TPW], si[TPW];
    {
      auto fa = [&](int i, int k) -> double2 {
        return cconj(B[i][k]);
      };
      auto fb = [&](int k, int jj) -> double2 {
        return B[jj][k];
      };
#pragma unroll
      for (int q = 0; q < TPW; ++q) {
        const int tile = wv + q * NW;
        if (tile < tg * tg) cgemm_tile(16 * (tile / tg), 16 * (tile - (tile / tg) * tg), nB, nB, mB, fa, fb, sr[q], si[q]);
      }
    }
    auto tile_ij = [&](int q, int& ti, int& tj) {
      const int tile = wv + q * NW;
      ti = tile / tg;
      tj = tile - ti * tg;
      return tile < tg * tg;
    };
    __shared__ double2 prow[2][NMAX];  // pivot rows of the Cholesky steps, by step parity
    if (tid < 2 * NMAX) prow[tid / NMAX][tid % NMAX] = make_double2(0.0, 0.0);  // columns past nB stay zero
    // R rows in pivot order over the B region: Rs[j][c] = R(j, position of column c)
    double2 (*const Rs)[NMAX] = reinterpret_cast<double2 (*)[NMAX]>(Bmem);
    // Every wave keeps the Schur complement's diagonal, lane c holding entry c, and updates it
    // from each pivot row, so each wave finds the next pivot by itself (the same one in every
    // wave) and the owners of that row publish it right after their update: one barrier per step.
    double dg = 0.0;
    unsigned long long usedmask = 0ull;
    // column of the largest remaining diagonal entry.  The key is the entry's high word (sign,
    // exponent and 20 mantissa bits, in the order of the values for non-negative ones) with its 6
    // lowest bits replaced by 63 - column, 0 for a used, padded or non-positive entry: entries
    // within ~2^-14 of each other count as equal and the lowest column wins.  With every key 0 it
    // returns 63, whose diagonal copy is then not positive, so the caller's stop test ends.
    auto next_pivot = [&]() -> int {
      unsigned key = 0u;
      if (lane < nB && !((usedmask >> lane) & 1ull) && dg > 0.0)
        key = ((unsigned)__double2hiint(dg) & ~63u) | (unsigned)(63 - lane);
      return 63 - (int)(wave_umax_uniform(key) & 63u);
    };
    int j = 0;
    if constexpr (NMAX == 64) {
      // D <= 32: S stays in the Gram tiles' registers and the rank-1 updates of four steps are
      // applied together, as one complex rank-4 product per tile on the matrix cores.  Until
      // then each pending row i is kept in registers twice, as rl[i] = R_i[lane] (any column by
      // readlane) and rc[q][i] = R_i at the lane's column of tile q; the owners of the next pivot
      // row apply the pending rows to it before publishing it.
      __shared__ double diag[NMAX];
#pragma unroll
      for (int q = 0; q < TPW; ++q) {
        int ti, tj;
        if (tile_ij(q, ti, tj) && ti == tj && (li & 3) == lk) {
          const int r = li >> 2;
          diag[16 * ti + li] = r == 0 ? sr[q][0] : r == 1 ? sr[q][1] : r == 2 ? sr[q][2] : sr[q][3];
        }
      }
      __syncthreads();
      if (lane < nB) dg = diag[lane];
      double2 rl[4], rc[TPW][4];
      auto publish_row = [&](int P, int np, int buf) {
        double2 rp[4];  // R_i[P] of the pending rows
#pragma unroll
        for (int i = 0; i < 4; ++i)
          rp[i] = i < np ? make_double2(readlane_d(rl[i].x, P), readlane_d(rl[i].y, P)) : make_double2(0.0, 0.0);
        const int rr = P & 15, r4 = rr >> 2;
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
          int ti, tj;
          if (tile_ij(q, ti, tj) && ti == (P >> 4) && lk == (rr & 3)) {
            const int c = 16 * tj + li;
            double2 v = r4 == 0 ? make_double2(sr[q][0], si[q][0]) : r4 == 1 ? make_double2(sr[q][1], si[q][1])
                      : r4 == 2 ? make_double2(sr[q][2], si[q][2]) : make_double2(sr[q][3], si[q][3]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (i < np) v = csub(v, cmulc(rp[i], rc[q][i]));
            if (c < nB) prow[buf][c] = ((usedmask >> c) & 1ull) ? make_double2(0.0, 0.0) : v;
          }
        }
      };
      // the pivot, its diagonal value dP (lane copy) and 1 / sqrt(dP), ready before the barrier
      int P = next_pivot();
      double dP = readlane_d(dg, P);
      const double stop = dP * (64.0 * 2.220446049250313e-16);
      double rd = rsq_nr(dP);
      if (dP > stop) publish_row(P, 0, 0);
      __syncthreads();
      bool done = false;
      for (int jb = 0; !done; jb += 4) {
        if (jb > 0) {
          // S -= sum over the rows jb - 4 .. jb - 1 of conj(R_i[r]) R_i[c] (rows visible in LDS)
#pragma unroll
          for (int q = 0; q < TPW; ++q) {
            int ti, tj;
            if (tile_ij(q, ti, tj)) {
              const double2 a = Rs[jb - 4 + lk][16 * ti + li], b = Rs[jb - 4 + lk][16 * tj + li];
              sr[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.x, b.x, sr[q], 0, 0, 0);
              sr[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, sr[q], 0, 0, 0);
              si[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.x, b.y, si[q], 0, 0, 0);
              si[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, si[q], 0, 0, 0);
            }
          }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (j >= nB || !(dP > stop)) {  // the remaining Schur complement is rounding noise
            done = true;
            break;
          }
          const double2* pw = prow[j & 1];
          const double2 pv = pw[lane < NMAX ? lane : 0];  // first: the diagonal update waits only on it
          double2 pt[TPW];
#pragma unroll
          for (int q = 0; q < TPW; ++q) {
            int ti, tj;
            tile_ij(q, ti, tj);
            pt[q] = pw[(16 * tj + li) & (NMAX - 1)];
          }
          const double id = rd * rd;  // 1 / R(j, j)^2
          usedmask |= 1ull << P;
          dg = lane == P ? 0.0 : dg - cabs2(pv) * id;
          // row j of R, queued behind the reads (read after the barrier)
          rl[k] = cscale(pv, rd);
          if (tid == 0) colid[j] = P;
          if (tid < NMAX) Rs[j][tid] = tid >= nB ? make_double2(0.0, 0.0) : tid == P ? make_double2(dP * rd, 0.0) : rl[k];
          const int Pn = next_pivot();
          const double dPn = readlane_d(dg, Pn);
#pragma unroll
          for (int q = 0; q < TPW; ++q) rc[q][k] = cscale(pt[q], rd);
          ++j;
          if (j < nB && dPn > stop) publish_row(Pn, k + 1, j & 1);
          P = Pn;
          dP = dPn;
          rd = rsq_nr(dP);
          __syncthreads();
        }
      }
    } else {
      // D <= 16: the step is bound by its chain, not by issue: thread (br, bc) holds the E x E
      // block of rows br E.., columns bc E.. of S and applies every rank-1 update at once.
      constexpr int GB = NT == 256 ? 16 : 8;  // blocks per side
      constexpr int E = NMAX / GB;
      static_assert(GB * GB == NT && E * GB == NMAX, "Cholesky blocks");
      const int br = tid / GB, bc = tid - (tid / GB) * GB;
      __syncthreads();
      {
        double2 (*const Gs)[NMAX + 1] = reinterpret_cast<double2 (*)[NMAX + 1]>(Bmem);
#pragma unroll
        for (int q = 0; q < TPW; ++q) {
          int ti, tj;
          if (tile_ij(q, ti, tj)) {
#pragma unroll
            for (int r = 0; r < 4; ++r) Gs[16 * ti + lk + 4 * r][16 * tj + li] = make_double2(sr[q][r], si[q][r]);
          }
        }
      }
      __syncthreads();
      double2 g[E][E];
      {
        double2 (*const Gs)[NMAX + 1] = reinterpret_cast<double2 (*)[NMAX + 1]>(Bmem);
#pragma unroll
        for (int a = 0; a < E; ++a)
#pragma unroll
          for (int b = 0; b < E; ++b) {
            const int r = br * E + a, c = bc * E + b;
            const double2 t = Gs[r][c];
            g[a][b] = (r < nB && c < nB) ? t : make_double2(0.0, 0.0);
          }
        if (lane < nB) dg = Gs[lane][lane].x;
      }
      auto publish_row = [&](int P, int buf) {
        if (br == P / E) {
#pragma unroll
          for (int a = 0; a < E; ++a)
            if (br * E + a == P)
#pragma unroll
              for (int b = 0; b < E; ++b)
                if (bc * E + b < nB) prow[buf][bc * E + b] = g[a][b];
        }
      };
      int P = next_pivot();
      double dP = readlane_d(dg, P);
      const double stop = dP * (64.0 * 2.220446049250313e-16);
      double rd = rsq_nr(dP);
      if (dP > stop) publish_row(P, 0);
      __syncthreads();
      for (; j < nB; ++j) {
        if (!(dP > stop)) break;  // the remaining Schur complement is rounding noise
        const double2* pw = prow[j & 1];
        // every LDS read of the step is issued here, the pivot row entry of the lane's column
        // first: the diagonal update and the next pivot wait only on it
        const double2 pv = pw[lane < NMAX ? lane : 0];
        double2 pr[E], pc[E];
#pragma unroll
        for (int a = 0; a < E; ++a) {
          pr[a] = pw[br * E + a];
          pc[a] = pw[bc * E + a];
        }
        const double id = rd * rd;  // 1 / R(j, j)^2
        usedmask |= 1ull << P;
        dg = lane == P ? 0.0 : dg - cabs2(pv) * id;
        // row j of R, queued behind the reads
        if (tid == 0) colid[j] = P;
        if (tid < nB) Rs[j][tid] = tid == P ? make_double2(dP * rd, 0.0) : cscale(pv, rd);
        const int Pn = next_pivot();
        const double dPn = readlane_d(dg, Pn);
        // S[r][c] -= conj(S[P][r]) S[P][c] / S[P][P] (S Hermitian).  The rows and columns of the
        // pivots already taken keep rounding residue instead of zeros: no entry of R, no diagonal
        // entry left in play and no update of an entry left in play reads them.
#pragma unroll
        for (int a = 0; a < E; ++a) {
          const double2 ps = cscale(pr[a], id);
#pragma unroll
          for (int b = 0; b < E; ++b) {
            g[a][b].x = fma(-ps.x, pc[b].x, fma(-ps.y, pc[b].y, g[a][b].x));
            g[a][b].y = fma(-ps.x, pc[b].y, fma(ps.y, pc[b].x, g[a][b].y));
          }
        }
        if (dPn > stop) publish_row(Pn, (j + 1) & 1);
        P = Pn;
        dP = dPn;
        rd = rsq_nr(dP);
        __syncthreads();
      }
    }
    // never-pivoted columns (zero Schur complement) follow in ascending order
    if (tid == 0)
      for (int c = 0, k = j; c < nB; ++c)
        if (!((usedmask >> c) & 1ull)) colid[k++] = c;
    __syncthreads();
    // B <- R^H on the leading nB x nB block: X[c][r] = conj(R(c, r)) = conj(Rs[c][colid[r]]),
    // c <= r, rows of R past the last pivot zero
    double2 xt[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int idx = tid + e * NT;
      const int c = idx / nB, rr = idx - (idx / nB) * nB;
      xt[e] = (idx < nB * nB && c <= rr && c < j) ? cconj(Rs[c][colid[rr]]) : make_double2(0.0, 0.0);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      const int idx = tid + e * NT;
      const int c = idx / nB, rr = idx - (idx / nB) * nB;
      if (idx < nB * nB) B[c][rr] = xt[e];
    }
    __syncthreads();
  } else {
    // complex128 path: Householder QR of B, its columns in falling order of their norms.  Group c
    // (LQ lanes) holds the column of position c in registers; one barrier per column: the owner of
    // position j + 1 publishes its rows and their squared norm (below the diagonal) right after
    // reflector j, and every group rebuilds reflector j + 1 from that copy, bit-identically.  The
    // reflectors, scaled by sqrt(tau) (H = I - v v^H), are kept in the item's T buffer, which
    // nothing else uses before the T matrices are written.
    constexpr int LQ = NT / NMAX;
    constexpr int RQ = NMAX / LQ;
    __shared__ double2 vb[2][NMAX];
    __shared__ double vn[2];
    double2* const refl = reinterpret_cast<double2*>(st.tbuf) + rbuf_off(st, slot, 0, 0);  // [nB][mB]
    if (small_sq) {
      static_assert(kSmallB * kSmallB <= NT, "one entry per thread");
      const int c = tid / nB, rr = tid - (tid / nB) * nB;
      const bool in = tid < nB * nB;
      const double2 t = B[in ? rr : 0][in ? c : 0];
      __syncthreads();
      if (in) B[c][rr] = cconj(t);
      if (tid < nB) colid[tid] = tid;
      __syncthreads();
    } else {
    const int qc = tid / LQ, ql = tid - (tid / LQ) * LQ;
    const int qfirst = (__builtin_amdgcn_readfirstlane(tid) >> 6) * (64 / LQ);  // first column of this wave
    {
      double s2 = 0.0;
      if (qc < nB)
        for (int rr = ql; rr < mB; rr += LQ) s2 += cabs2(B[qc][rr]);
      s2 = group_sum_dpp(s2, LQ);
      if (ql == 0) nrm[qc] = qc < nB ? s2 : -1.0;
    }
    __syncthreads();
    if (tid < nB) colid[falling_rank(nrm, nB, tid)] = tid;
    __syncthreads();
    // RQB row blocks of LQ rows: a matrix of fewer rows leaves the others out.  A wave without columns,
    // or with none left, takes part in the barriers only.
    auto qr = [&](auto row_blocks) {
      constexpr int RQB = decltype(row_blocks)::value;
      double2 x[RQB];
#pragma unroll
      for (int u = 0; u < RQB; ++u) {
        const int rr = ql + LQ * u;
        x[u] = (qc < nB && rr < mB) ? B[colid[qc < nB ? qc : 0]][rr] : make_double2(0.0, 0.0);
      }
      auto publish = [&](int j) {  // rows and the norm below row j of the column of position j
        double s2 = 0.0;
#pragma unroll
        for (int u = 0; u < RQB; ++u) {
          const int rr = ql + LQ * u;
          vb[j & 1][rr] = x[u];
          if (rr > j) s2 += cabs2(x[u]);
        }
        s2 = group_sum_dpp(s2, LQ);
        if (ql == 0) vn[j & 1] = s2;
      };
      if (qc == 0) publish(0);
      __syncthreads();
      for (int j = 0; j < nB; ++j) {
        if (qfirst >= nB || qfirst + 64 / LQ <= j) {
          __syncthreads();
          continue;
        }
        const double2 alpha = vb[j & 1][j];
        const double s2 = vn[j & 1];
        double2 v[RQB];
#pragma unroll
        for (int u = 0; u < RQB; ++u) v[u] = vb[j & 1][ql + LQ * u];
        // reflector v = x - beta e_j, beta = -phase(x_j) ||x||, x = rows j.. of the column; an exactly
        // zero lower part needs none
        const bool any = s2 > 0.0;
        const double aa2 = cabs2(alpha);
        const double nu2 = any ? aa2 + s2 : 1.0;
        const double nu = nu2 * rsq_nr(nu2);
        const double2 ph = aa2 > 0.0 ? cscale(alpha, rsq_nr(aa2)) : make_double2(1.0, 0.0);
        const double2 beta = any ? cscale(ph, -nu) : alpha;
        const double2 v0 = csub(alpha, beta);
        const double tau = any ? 2.0 * rcp_nr(cabs2(v0) + s2) : 0.0;
#pragma unroll
        for (int u = 0; u < RQB; ++u) {
          const int rr = ql + LQ * u;
          v[u] = rr == j ? v0 : rr > j ? v[u] : make_double2(0.0, 0.0);
        }
        if (qc > j && qc < nB) {
          double wr = 0.0, wi = 0.0;
#pragma unroll
          for (int u = 0; u < RQB; ++u) {
            const double2 t = cmulc(v[u], x[u]);
            wr += t.x;
            wi += t.y;
          }
          group_sum2_dpp(wr, wi, LQ);
          const double2 f = make_double2(wr * tau, wi * tau);
#pragma unroll
          for (int u = 0; u < RQB; ++u) x[u] = csub(x[u], cmul(v[u], f));
          if (qc == j + 1) publish(j + 1);
        } else if (qc == j) {
          const double rt = any ? tau * rsq_nr(tau) : 0.0;
#pragma unroll
          for (int u = 0; u < RQB; ++u) {
            const int rr = ql + LQ * u;
            if (rr < mB) refl[j * mB + rr] = cscale(v[u], rt);
            if (rr == j) x[u] = beta;
          }
        }
        __syncthreads();
      }
      // B <- R^H: X[c][r] = conj(R(c, r)), c <= r, from the registers of column r
#pragma unroll
      for (int u = 0; u < RQB; ++u) {
        const int c = ql + LQ * u;
        if (qc < nB && c < nB) B[c][qc] = c <= qc ? cconj(x[u]) : make_double2(0.0, 0.0);
      }
    };
    if (mB <= LQ * RQ / 4) qr(std::integral_constant<int, RQ / 4>());
    else if (mB <= LQ * RQ / 2) qr(std::integral_constant<int, RQ / 2>());
    else qr(std::integral_constant<int, RQ>());
    __syncthreads();
    }
  }

  constexpr int LJ = 2 * NT / NMAX;  // lanes per column pair
  const int pair_id = tid / LJ;
  const int lane = tid - pair_id * LJ;
  // lane `lane` holds rows lane + LJ ((u + jsh) mod RPL); when several pairs share a 16-lane LDS
  // cycle (LJ < 16) they start on consecutive row blocks, so their accesses use disjoint banks
  constexpr int PW = LJ < 16 ? 16 / LJ : 1;  // pairs per 16-lane group
  static_assert((RPL & (RPL - 1)) == 0 && RPL >= PW, "Jacobi row blocks");
  const int jsh = pair_id & (PW - 1);
  auto jrow = [&](int u) { return lane + LJ * ((u + jsh) & (RPL - 1)); };
  const double tol2 = (2.220446049250313e-16 * (double)nB) * (2.220446049250313e-16 * (double)nB);
  int sweep = 0;
  bool converged = (nB < 2);
  {
    // Register-resident Jacobi on X = R^H (nB x nB).  The columns are padded to
    // 2^K >= nB and paired as {c, c ^ m} for m = 1 .. 2^K - 1, a complete sweep in which every
    // round is a perfect matching.  The rounds run in blocks of equal highest bit hb of m: inside
    // a block the column of the pair with bit hb clear stays in the registers of its lane group
    // g = c with bit hb deleted, and its partner (bit hb set) sits in group
    // g = (c ^ m) with bit hb deleted.  Between rounds the moving columns change groups so that
    // each visits every stationary one of its block once.  GW = 64 / LJ groups share a wave:
    //   LJ = 16: the lanes of a group are consecutive (its sums are four DPP levels, the shortest
    // chain: this size is bound by latency), and the low bits m' of m go through a Gray code,
    // so that a column moves by lane ^ 16 or ^ 32 (v_permlane swaps);
    //   LJ = 8, 4: the lanes of a group are spread over l / 16, the group index inside the wave is
    // (blk, low), blk in lane bits 2 and 3, low in the upper bits of the lane's quad.  low walks
    // through a Gray code (DPP quad permutation), blk rotates (DPP row_ror:4): one DPP instruction
    // a word, 5.5 cycles of issue against 8.6 of a v_permlane swap, and the moves are most of the
    // words.  In blocks of fewer than GW rounds blk moves by lane ^ 4.
    // After GW rounds the columns pass to the wave whose index differs in one bit (Gray code)
    // through LDS.  Between blocks (and at the end of every sweep) all columns are written to B
    // and re-read under the next block's assignment.  With ACC the columns of W travel with
    // those of X.
    //   The rotation of smaller angle (|theta| <= pi/4) with tan 2 theta = 2|g| / (be - al):
    // h = (d^2 + 4|g|^2)^1/2, d = be - al, x = cos^2 theta = (1 + |d| / h) / 2; |g| itself is never
    // formed.
    //   LJ = 16: c = x^1/2 and s e^{i phi} = sign(d) g / (h x^1/2), the shorter chain.
    //   LJ = 8, 4 (more rows a lane, bound by issue): tan theta e^{i phi} = g F, F = sign(d) / (h x),
    // and the columns carry a scale: the column is sqrt(ps) xs, a rotation is
    // xs -= conj(g F) pm xm, xm += g F ps xs (g the inner product of the scaled columns) with both
    // squared scales times x: 8 instead of 12 operations per complex pair of entries.  The scales
    // are folded in at the start of a sweep and after the last one.  The inner products are summed
    // with v_mfma_f64_4x4x4_4b_f64 against ones (lane l supplies A[l % 4][l / 16] and
    // B[l / 16][l % 4] of block (l / 4) % 4 and receives D[l / 16][l % 4]).
    //   32 instances at D = 32, per launch: 1188 us with the LJ = 16 forms at LJ = 8, 1186 with the
    // sums on the matrix cores alone, 1164 with the scales alone, 1138 with both (101.9 k cycles a
    // sweep of 63 rounds, two workgroups a CU).  At D = 16, one instance, the LJ = 8 forms took
    // 87.7 us against 83.
    constexpr int GW = 64 / LJ;                         // lane groups per wave
    constexpr int LB = LJ == 16 ? 0 : LJ == 8 ? 1 : 2;  // bits of low
    constexpr bool kSpread = LJ != 16;
    static_assert(GW == 4 << LB, "lane groups");
    const int wl = tid & 63;
    const int jgrp = kSpread ? (tid >> 6) * GW + ((((wl >> 2) & 3) << LB) | ((wl & 3) >> (2 - LB))) : tid / LJ;
    const int jlane = kSpread ? (wl & ((4 >> LB) - 1)) + (4 >> LB) * (wl >> 4) : tid & (LJ - 1);
    const double own = ((wl >> 4) >> 1) == ((wl & 3) >> 1) ? 1.0 : 0.0;  // LJ = 8: the two groups of a block apart
    int K = 1;
    while ((1 << K) < nB) ++K;
    const bool gact = jgrp < (1 << (K - 1));
    auto ins = [](int g, int hb, int bit) { return ((g >> hb) << (hb + 1)) | (bit << hb) | (g & ((1 << hb) - 1)); };
    auto xrow = [&](int u) { return jlane + LJ * u; };
    auto group_total2 = [&](double& a, double& b, int rows) {
      if constexpr (!kSpread) {
        group_sum2_dpp(a, b, rows < LJ ? rows : LJ);
      } else {
        if constexpr (LJ == 8) {
          a = own * __builtin_amdgcn_mfma_f64_4x4x4f64(a, 1.0, 0.0, 0, 0, 0);  // sum over l / 16 of l % 4 = i, in D[i][j]
          b = own * __builtin_amdgcn_mfma_f64_4x4x4f64(b, 1.0, 0.0, 0, 0, 0);
        }
        a = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, a, 0.0, 0, 0, 0);
        b = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, b, 0.0, 0, 0, 0);
      }
    };
    // per-sweep flags (any rotation, any rotation above the quiet level), three sets in
    // rotation so that a set is cleared neither while it is read nor after it is written
    __shared__ int sh_flag[3][2];
    if (tid < 6) sh_flag[tid >> 1][tid & 1] = 0;
    // the padding columns (ids nB .. 2^K - 1) and the ids of inactive groups are exactly zero:
    // their tracked norms are zero too (store_col never writes them), which keeps the rotation
    // scalars of every pair finite
    for (int c = nB + tid; c < NMAX; c += NT) nrm[c] = 0.0;
    if (kSpread)
      for (int c = tid; c < NMAX; c += NT) scl[c] = 1.0;
    __syncthreads();
    // RB row blocks of LJ rows: a matrix of at most half the rows leaves the upper half of them out.
    // SOLO: at most 8 columns, LJ = 16 lanes a pair: one wave has them all, goes without barriers and sums over
    // the lanes that have rows; the others wait for it (24-qubit ring, 6 columns: 31 -> 29 us a launch).
    auto sweeps = [&](auto row_blocks, auto solo) {
      constexpr int RB = decltype(row_blocks)::value;
      constexpr bool SOLO = decltype(solo)::value;
      constexpr int SR = SOLO ? 8 : 64;  // rows of a sum
      auto barrier = [&]() {
        if constexpr (SOLO) wave_lds_sync();
        else __syncthreads();
      };
      if (SOLO && __builtin_amdgcn_readfirstlane(tid) >= 64) return;
      // a wave whose groups are all inactive takes part in the barriers only (uniform over the wave;
      // with every row block at NMAX = 64 none is, and the test costs 0.7 %); complex128 up to D = 16 leaves
      // out every GW rounds in which a wave has none of the nB columns to move, too: 18 columns run as
      // 32, and with several workgroups a CU the rounds on padding cost what they issue (127 qubits x 16 at
      // D = 9, 12 steps 9.90 -> 8.24 ms)
      const int wgrp = (__builtin_amdgcn_readfirstlane(tid) >> 6) * GW;  // first group of this wave
      const bool wact = (NMAX == 64 && RB == RPL) || wgrp < (1 << (K - 1));
      auto moves = [&](int hb, int t0) {  // of rounds t0 .. t0 + GW - 1 of block hb
        if constexpr (ACC && NMAX == 32) return ins(wgrp ^ ((t0 ^ (t0 >> 1)) & ~(GW - 1)), hb, 1) < nB;
        else return wact;
      };
      double2 xs[RB], xm[RB];  // stationary and moving column of the group
      double2 us[ACC ? RB : 1], um[ACC ? RB : 1];  // and the columns of W that go with them
      double ns = 0.0, nm = 0.0;  // their tracked squared norms
      double ps = 1.0, pm = 1.0;  // their squared scales
      int cs_id = 0, cm_id = 0;   // their column indices
      auto load_col = [&](double2 (&x)[RB], double2 (&w)[ACC ? RB : 1], int c) {
#pragma unroll
        for (int u = 0; u < RB; ++u) {
          const int rr = xrow(u);
          const double2 t = B[c][rr];
          x[u] = (gact && c < nB && rr < nB) ? t : make_double2(0.0, 0.0);
          if constexpr (ACC) {
            const double2 q = W[c][rr];
            w[u] = (gact && c < nB && rr < nB) ? q : make_double2(0.0, 0.0);
          }
        }
      };
      auto store_col = [&](const double2 (&x)[RB], const double2 (&w)[ACC ? RB : 1], int c, double n2, double p2) {
        if (gact && c < nB) {
#pragma unroll
          for (int u = 0; u < RB; ++u) {
            const int rr = xrow(u);
            if (rr < nB) {
              B[c][rr] = x[u];
              if constexpr (ACC) W[c][rr] = w[u];
            }
          }
          if (jlane == 0) {
            nrm[c] = n2;
            if (kSpread) scl[c] = p2;
          }
        }
      };
      // the scale of a column folded in: its squared norm, with the scale back at 1
      auto fold = [&](double2 (&x)[RB], double2 (&w)[ACC ? RB : 1], double& p2) {
        if constexpr (kSpread) {
          const double d = p2 * rsq_nr(p2);
#pragma unroll
          for (int u = 0; u < RB; ++u) {
            x[u] = cscale(x[u], d);
            if constexpr (ACC) w[u] = cscale(w[u], d);
          }
          p2 = 1.0;
        }
        double s2 = 0.0;
#pragma unroll
        for (int u = 0; u < RB; ++u) s2 += cabs2(x[u]);
        return s2;
      };
      bool rot = false, big = false;
      const double floor2 = sh_floor * sh_floor;
      for (; sweep < st.max_sweeps && !converged; ++sweep) {
        for (int hb = 0; hb < K; ++hb) {
          cs_id = ins(jgrp, hb, 0);
          cm_id = ins(jgrp, hb, 1);
          load_col(xs, us, cs_id);
          load_col(xm, um, cm_id);
          if (kSpread) {
            ps = scl[cs_id];
            pm = scl[cm_id];
          }
          if (hb == 0) {
            ns = fold(xs, us, ps);
            nm = fold(xm, um, pm);
            group_total2(ns, nm, SR);
          } else {
            ns = nrm[cs_id];
            nm = nrm[cm_id];
          }
          const int nt = 1 << hb;
          // the moving column (with its norm and scale where the columns carry one) through one lane
          // permutation
          auto move = [&](auto perm2) {
#pragma unroll
            for (int u = 0; u < RB; ++u) {
              perm2(xm[u].x, xm[u].y);
              if constexpr (ACC) perm2(um[u].x, um[u].y);
            }
            if constexpr (kSpread) perm2(nm, pm);
          };
          auto move_low = [&](int bit) {  // low ^ 2^bit
            if (LB == 2 && bit == 0) move([](double& a, double& b) { a = dpp_d<0xB1>(a); b = dpp_d<0xB1>(b); });  // lane ^ 1
            else move([](double& a, double& b) { a = dpp_d<0x4E>(a); b = dpp_d<0x4E>(b); });                      // lane ^ 2
          };
          auto move_xor = [&](int bit) {  // blocks of fewer than GW rounds, and LJ = 16: group ^ 2^bit
            if constexpr (!kSpread) {
              if (bit == 0) {
                move([](double& a, double& b) { lane_xor_pair<16>(a, b); });
                nm = lane_xor<16>(nm);
              } else {
                move([](double& a, double& b) { lane_xor_pair<32>(a, b); });
                nm = lane_xor<32>(nm);
              }
            } else if (bit < LB) {
              move_low(bit);
            } else {
              move([](double& a, double& b) { a = lane_xor<4>(a); b = lane_xor<4>(b); });
            }
          };
          auto move_blk = [&](int sb) {
            if constexpr (!kSpread) move_xor(sb & 1);  // bits 0, 1, 0
            else move([](double& a, double& b) { a = dpp_d<0x124>(a); b = dpp_d<0x124>(b); });  // blk - 1 to blk
          };
          // one round: the rotation of the group's pair (stationary xs, moving xm).  Branch-free:
          // a pair that is not rotated takes F = 0, x = 1 (s = 0, c = 1), which leaves both columns and
          // norms bit for bit.  Padding columns are exactly zero, so their pairs have g = 0 and are
          // never rotated; h is kept away from zero so that every pair's scalars stay finite.
          auto round = [&]() {
            double gr, gi;
            if constexpr (RB >= 4) {
              dot_rows<RB>(xs, xm, gr, gi);
            } else {  // the shorter chain
              double2 g = cmulc(xs[0], xm[0]);
#pragma unroll
              for (int u = 1; u < RB; ++u) g = cadd(g, cmulc(xs[u], xm[u]));
              gr = g.x;
              gi = g.y;
            }
            group_total2(gr, gi, SR);
            const double al = ns, be = nm;
            const double g2 = kSpread ? (gr * gr + gi * gi) * (ps * pm) : gr * gr + gi * gi;
            const double ab = al * be;
            const bool ok = (g2 > tol2 * ab) & (g2 > floor2);
            const double d = be - al;
            const double h2 = fmax(d * d + 4.0 * g2, 1e-300);
            const double rh = ACC ? rsq_nr(h2) : rsq_nr1(h2);  // 1 / h
            const double x = 0.5 + 0.5 * fabs(d) * rh;
            double tg, t2 = 0.0;  // tan theta |g|, tan^2 theta
            if constexpr (kSpread) {
              const double rx = ACC ? rcp_nr(x) : rcp_nr1(x);  // 1 / x
              const double F = ok ? copysign(rh, d) * rx : 0.0;
              const double xx = ok ? x : 1.0;
              tg = g2 * F;
              if constexpr (ACC) t2 = tg * F;
              const double fm = F * pm, fs = F * ps;
              const double2 tm = make_double2(gr * fm, gi * fm), ts = make_double2(gr * fs, gi * fs);
              auto turn = [&](double2& a, double2& b) {
                const double2 a0 = a;
                a.x = fma(-tm.x, b.x, fma(-tm.y, b.y, a.x));
                a.y = fma(-tm.x, b.y, fma(tm.y, b.x, a.y));
                b.x = fma(ts.x, a0.x, fma(-ts.y, a0.y, b.x));
                b.y = fma(ts.x, a0.y, fma(ts.y, a0.x, b.y));
              };
#pragma unroll
              for (int u = 0; u < RB; ++u) {
                turn(xs[u], xm[u]);
                if constexpr (ACC) turn(us[u], um[u]);
              }
              ps *= xx;
              pm *= xx;
            } else {
              const double rc = ACC ? rsq_nr(x) : rsq_nr1(x);  // 1 / c
              const double f = ok ? copysign(rh, d) * rc : 0.0;
              const double cs = ok ? x * rc : 1.0;
              const double2 sph = make_double2(gr * f, gi * f);  // s e^{i phi}
              if constexpr (ACC) {
                const double F = f * rc;
                tg = g2 * F;
                t2 = tg * F;
              } else {
                tg = g2 * f * rc;
              }
              auto turn = [&](double2& a, double2& b) {
                const double2 a0 = a, b0 = b;
                a = csub(cscale(a0, cs), cmulc(sph, b0));
                b = cadd(cmul(sph, a0), cscale(b0, cs));
              };
#pragma unroll
              for (int u = 0; u < RB; ++u) {
                turn(xs[u], xm[u]);
                if constexpr (ACC) turn(us[u], um[u]);
              }
            }
            ns = al - tg;
            nm = be + tg;
            rot |= ok;
            big |= ok & ((g2 > (ACC ? kJacobiQuietC128 : kJacobiQuietC64) * ab) | (ACC && t2 > kJacobiQuietC128));
          };
          // the moving column of this group in round t of the block
          auto mid = [&](int t) {
            if (!kSpread || nt < GW) return ins(jgrp ^ (t ^ (t >> 1)), hb, 1);
            constexpr int ML = (1 << LB) - 1;  // low's Gray code ends at its last value, where the next one starts
            const int T = t / GW, sb = (t >> LB) & 3, r = t & ML;
            const int low = (jgrp & ML) ^ (r ^ (r >> 1)) ^ ((sb & 1) ? (ML ^ (ML >> 1)) : 0);
            const int blk = (((jgrp >> LB) & 3) - sb) & 3;
            const int w = (jgrp / GW) ^ (T ^ (T >> 1));
            return ins((w * 4 + blk) << LB | low, hb, 1);
          };
          if (nt < GW) {
            if (moves(hb, 0)) {
              for (int t = 0; t < nt; ++t) {
                round();
                if (t + 1 < nt) move_xor(__builtin_ctz(t + 1));
              }
            }
          } else {
            // (spread lanes: blk turns once more than it has to, so that every trip is the same
            // straight line and the columns end where they began the GW rounds)
            for (int t0 = 0; t0 < nt; t0 += GW) {
              if (moves(hb, t0)) {
                auto quarter = [&](int sb) {
#pragma unroll
                  for (int r = 0; r < 1 << LB; ++r) {
                    round();
                    if (r + 1 < 1 << LB) move_low(__builtin_ctz(r + 1));
                  }
                  if (kSpread || sb < 3) move_blk(sb);
                };
                if constexpr (RB >= 8 || NMAX == 64) {  // straight-line code of that length takes the compiler many minutes
#pragma unroll 1
                  for (int sb = 0; sb < 4; ++sb) quarter(sb);
                } else {
#pragma unroll
                  for (int sb = 0; sb < 4; ++sb) quarter(sb);
                }
              }
              if (t0 + GW < nt) {
                store_col(xm, um, mid(kSpread ? t0 : t0 + GW - 1), nm, pm);
                barrier();
                load_col(xm, um, mid(t0 + GW));
                nm = nrm[mid(t0 + GW)];
                if (kSpread) pm = scl[mid(t0 + GW)];
              }
            }
          }
          cm_id = mid(kSpread && nt >= GW ? nt - GW : nt - 1);
          // end of the block: every column back to B (with its tracked norm and scale)
          store_col(xs, us, cs_id, ns, ps);
          store_col(xm, um, cm_id, nm, pm);
          if (hb + 1 == K) {
            if (rot && jlane == 0) sh_flag[sweep % 3][0] = 1;
            if (big && jlane == 0) sh_flag[sweep % 3][1] = 1;
            if (tid < 2) sh_flag[(sweep + 1) % 3][tid] = 0;
            rot = false;
            big = false;
          }
          barrier();
        }
        converged = (sh_flag[sweep % 3][0] == 0) || (sh_flag[sweep % 3][1] == 0);
      }
    };
    if constexpr (NMAX == 64 && ACC) {
      // the first steps above D = 16 (one 24-qubit ring, D = 20, launch of 4 / 8 / 16 / 32 columns: all eight row
      // blocks 33 / 91 / 155 / 262 us, these 21 / 42 / 74 / 188)
      if (nB <= 2 * LJ) sweeps(std::integral_constant<int, 2>(), std::false_type());
      else if (nB <= 4 * LJ) sweeps(std::integral_constant<int, 4>(), std::false_type());
      else sweeps(std::integral_constant<int, RPL>(), std::false_type());
    } else {
      constexpr int kHalf = NMAX == 32 ? RPL / 2 : RPL;
      constexpr bool kSolo = ACC && LJ == 16;
      if (kHalf == RPL || nB > LJ * kHalf) sweeps(std::integral_constant<int, RPL>(), std::false_type());
      else if (!kSolo || nB > 8) sweeps(std::integral_constant<int, kHalf>(), std::false_type());
      else sweeps(std::integral_constant<int, kHalf>(), std::integral_constant<bool, kSolo>());
      if (kSolo && nB <= 8) __syncthreads();
    }
  }
  if (tid == 0) count_svd(st, sweep, converged);

  // singular values (column norms, two columns per pair group, the scales folded in), stable
  // descending order
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int c = 2 * pair_id + h;
    const double d = LJ != 16 ? scl[c] * rsq_nr(scl[c]) : 1.0;
    double s2 = 0.0;
#pragma unroll
    for (int u = 0; u < RPL; ++u) {
      const int rr = jrow(u);
      double2 t = B[c][rr];
      if (c < nB && rr < nB) {
        if constexpr (LJ != 16) {
          t = cscale(t, d);
          B[c][rr] = t;
          if constexpr (ACC) W[c][rr] = cscale(W[c][rr], d);
        }
        s2 += cabs2(t);
      }
    }
    s2 = group_sum_dpp(s2, LJ);
    if (lane == 0 && c < nB) sig[c] = sqrt(s2);
  }
  __syncthreads();
  for (int c = tid; c < nB; c += NT) perm[falling_rank(sig, nB, c)] = c;
  __syncthreads();
  // truncation (one wave; nB <= 64): chi = #{sigma > trunc_rel sigma_0} capped at D (at least
  // 1), and the norm of the kept values for lambda_e
  if (tid < 64) {
    const double smax = sig[perm[0]];
    const int keep = __popcll(__ballot(tid < nB && sig[tid] > st.trunc_rel * smax));
    int chi = keep < D ? keep : D;
    if (chi < 1) chi = 1;
    const double sk = tid < chi ? sig[perm[tid]] : 0.0;
    const double nr = sqrt(group_sum_dpp(sk * sk, 64));
    if (tid == 0) {
      if (!(smax > 0.0)) flag_status(st.status, kStatusZeroTheta);
      if (!isfinite(nr)) flag_status(st.status, kStatusNonFinite);
      sh_chi = chi;
      sh_norm = nr;
      st.meta[slot].de_old = de;
      st.meta[slot].chi_new = chi;
      st.chi[e] = chi;
    }
  }
  __syncthreads();
  const int chi = sh_chi;
  for (int k = tid; k < D; k += NT) lam_e[k] = k < chi ? sig[perm[k]] / sh_norm : 0.0;
  if (BWD) {
    // every singular triplet: U [m0 x r], V [n0 x r], S [r], r = nB, row stride 2D; vectors
    // with sigma <= 1e-13 sigma_0 are set to zero (the null space)
    const int ld = 2 * D;
    double2* Ug = st.bU + (int64_t)slot * ld * ld;
    double2* Vg = st.bV + (int64_t)slot * ld * ld;
    const double smax = sig[perm[0]];
    for (int k = tid; k < nB; k += NT) st.bS[(int64_t)slot * ld + k] = sig[perm[k]];
    {
      // the Jacobi side is B's right singular vectors (rows permuted by the ordering), i.e. V of
      // Theta' when B = Theta', U when B = Theta'^H
      for (int idx = tid; idx < nB * nB; idx += NT) {
        const int rr = idx / nB, k = idx - (idx / nB) * nB;
        const double sv = sig[perm[k]];
        const double2 bv = sv > 1e-13 * smax ? cscale(B[perm[k]][rr], 1.0 / sv) : make_double2(0.0, 0.0);
        (trans ? Ug : Vg)[colid[rr] * ld + k] = bv;
      }
    }
  }

  // complex128 path: Q W, the left singular vectors of B, in registers: group kc (LC lanes) takes
  // column kc of the sorted order (and, for the reverse sweep, kc + DM before it) and applies the
  // reflectors, last one first.  Done before the T matrices take the reflectors' place.
  constexpr int LC = NT / DM;
  constexpr int RC = NMAX / LC;
  const int kc = tid / LC, lc = tid - (tid / LC) * LC;
  double2 qw[ACC ? RC : 1];
  if constexpr (ACC) {
    const double2* const refl = reinterpret_cast<const double2*>(st.tbuf) + rbuf_off(st, slot, 0, 0);
#pragma unroll
    for (int u = 0; u < RC; ++u) qw[u] = make_double2(0.0, 0.0);
    const int kfirst = (__builtin_amdgcn_readfirstlane(tid) >> 6) * (64 / LC);  // first column of this wave
    auto left = [&](auto row_blocks, int batch) {  // (row blocks as in the QR)
      constexpr int RCB = decltype(row_blocks)::value;
      const int k = kc + batch * DM;
      const int col = perm[k < nB ? k : 0];
#pragma unroll
      for (int u = 0; u < RCB; ++u) {
        const int rr = lc + LC * u;
        const double2 t = W[col][rr];
        qw[u] = (k < nB && rr < nB) ? t : make_double2(0.0, 0.0);
      }
      double2 nv[RCB];  // the next reflector, in flight
      auto fetch = [&](int j) {
#pragma unroll
        for (int u = 0; u < RCB; ++u) {
          const int rr = lc + LC * u;
          nv[u] = rr < mB ? refl[j * mB + rr] : make_double2(0.0, 0.0);
        }
      };
      const int nr = small_sq ? 0 : nB;
      if (nr) fetch(nr - 1);
      for (int j = nr - 1; j >= 0; --j) {
        double2 v[RCB];
#pragma unroll
        for (int u = 0; u < RCB; ++u) v[u] = nv[u];
        if (j > 0) fetch(j - 1);
        double wr = 0.0, wi = 0.0;
#pragma unroll
        for (int u = 0; u < RCB; ++u) {
          const double2 t = cmulc(v[u], qw[u]);
          wr += t.x;
          wi += t.y;
        }
        group_sum2_dpp(wr, wi, LC);
        const double2 f = make_double2(wr, wi);
#pragma unroll
        for (int u = 0; u < RCB; ++u) qw[u] = csub(qw[u], cmul(v[u], f));
      }
      if (BWD && k < nB) {
        const int ld = 2 * D;
        double2* Og = (trans ? st.bV : st.bU) + (int64_t)slot * ld * ld;
#pragma unroll
        for (int u = 0; u < RCB; ++u) {
          const int rr = lc + LC * u;
          if (rr < mB) Og[rr * ld + k] = qw[u];
        }
      }
    };
    for (int batch = BWD ? 1 : 0; batch >= 0; --batch) {
      if (kfirst + batch * DM >= (BWD ? nB : chi)) continue;
      if (mB <= LC * RC / 2) left(std::integral_constant<int, RC / 2>(), batch);
      else left(std::integral_constant<int, RC>(), batch);
    }
    __syncthreads();  // every reflector has been read
  }

  CT* T = reinterpret_cast<CT*>(st.tbuf);
  CT* const Ti0 = T + rbuf_off(st, slot, 0, 0);
  CT* const Ti1 = T + rbuf_off(st, slot, 0, 1);
  CT* const Tj0 = T + rbuf_off(st, slot, 1, 0);
  CT* const Tj1 = T + rbuf_off(st, slot, 1, 1);
  // zero columns k' >= chi of every T (rows k < de)
  for (int idx = tid; idx < 4 * de * (D - chi); idx += NT) {
    const int w = idx / (de * (D - chi));
    const int rem = idx - w * de * (D - chi);
    const int k = rem / (D - chi), kp = chi + rem - (rem / (D - chi)) * (D - chi);
    if (BWD) st.t64[rbuf_off(st, slot, w >> 1, w & 1) + k * D + kp] = make_double2(0.0, 0.0);
    T[rbuf_off(st, slot, w >> 1, w & 1) + k * D + kp] = from_d2<CT>(make_double2(0.0, 0.0));
  }
  const double2 g00 = gate_phase(ip, 0, 0), g01 = gate_phase(ip, 0, 1);
  const double2 g10 = gate_phase(ip, 1, 0), g11 = gate_phase(ip, 1, 1);
  // T_w[k][k'] (w = 0, 1: end i slices; 2, 3: end j slices), float64 in the reverse sweep
  auto putT = [&](int w, int k, int kp, double2 v) {
    if (BWD) st.t64[rbuf_off(st, slot, w >> 1, w & 1) + k * D + kp] = v;
    T[rbuf_off(st, slot, w >> 1, w & 1) + k * D + kp] = from_d2<CT>(v);
  };

  if (ACC) {
    // both vector sets into the arenas: B's right vectors from the orthogonalised columns (rows
    // permuted by the ordering), its left ones from Q W
    double2 uv[RPT];
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
      const int idx = tid + u * NT;
      uv[u] = make_double2(0.0, 0.0);
      if (idx < nB * chi) {
        const int rr = idx / chi, kp = idx - (idx / chi) * chi;
        uv[u] = cscale(B[perm[kp]][rr], 1.0 / sig[perm[kp]]);
      }
    }
    __syncthreads();
    double2* Ul = A0;  // U [(s,a)][k'], row stride DS
    double2* Vl = Wmem;  // V [(t,b)][k'], row stride DS
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
      const int idx = tid + u * NT;
      if (idx < nB * chi) {
        const int rr = idx / chi, kp = idx - (idx / chi) * chi;
        (trans ? Ul : Vl)[colid[rr] * DS + kp] = uv[u];
      }
    }
#pragma unroll
    for (int u = 0; u < RC; ++u) {
      const int rr = lc + LC * u;
      if (kc < chi && rr < mB) (trans ? Vl : Ul)[rr * DS + kc] = qw[u];
    }
    __syncthreads();
    stage_r(A1, 0, ri);
    stage_r(Wmem + 2 * DM * DS, 1, rj);
    __syncthreads();
    const double2* RIl = A1;
    const double2* RJl = Wmem + 2 * DM * DS;
    for (int idx = tid; idx < de * chi; idx += NT) {
      const int k = idx / chi, kp = idx - (idx / chi) * chi;
      double2 x0 = make_double2(0.0, 0.0), x1 = x0, y0 = x0, y1 = x0;
      for (int b = 0; b < rj; ++b) {
        x0 = cadd(x0, cmul(RJl[b * DS + k], Vl[b * DS + kp]));
        x1 = cadd(x1, cmul(RJl[DM * DS + b * DS + k], Vl[(rj + b) * DS + kp]));
      }
      for (int a2 = 0; a2 < ri; ++a2) {
        y0 = cadd(y0, cmulc(Ul[a2 * DS + kp], RIl[a2 * DS + k]));
        y1 = cadd(y1, cmulc(Ul[(ri + a2) * DS + kp], RIl[DM * DS + a2 * DS + k]));
      }
      const double f = lam_old[k] / sig[perm[kp]];
      const double2 ti0 = cscale(cadd(cmul(g00, x0), cmul(g01, x1)), f);
      const double2 ti1 = cscale(cadd(cmul(g10, x0), cmul(g11, x1)), f);
      const double2 tj0 = cscale(cadd(cmul(g00, y0), cmul(g10, y1)), f);
      const double2 tj1 = cscale(cadd(cmul(g01, y0), cmul(g11, y1)), f);
      if (BWD) {
        double2* T64 = st.t64 + rbuf_off(st, slot, 0, 0);
        T64[0 * D * D + k * D + kp] = ti0;
        T64[1 * D * D + k * D + kp] = ti1;
        T64[2 * D * D + k * D + kp] = tj0;
        T64[3 * D * D + k * D + kp] = tj1;
      }
      {
        Ti0[k * D + kp] = from_d2<CT>(ti0);
        Ti1[k * D + kp] = from_d2<CT>(ti1);
        Tj0[k * D + kp] = from_d2<CT>(tj0);
        Tj1[k * D + kp] = from_d2<CT>(tj1);
      }
    }
    return;
  }

  // complex64 path: the Jacobi side from B, the other side through small products with the R
  // factors.  After preconditioning the Jacobi side is B's right singular vectors: V of Theta'
  // when B = Theta', U of Theta' when B = Theta'^H, so the orientation below is flipped.
  const bool vside = !trans;  // the Jacobi side holds V (rows (t,b)) rather than U (rows (s,a))
  {
    double2 v[RPT];
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
      const int idx = tid + u * NT;
      v[u] = make_double2(0.0, 0.0);
      if (idx < nB * chi) {
        const int rr = idx / chi, kp = idx - (idx / chi) * chi;
        v[u] = cscale(B[perm[kp]][rr], 1.0 / sig[perm[kp]]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
      const int idx = tid + u * NT;
      if (idx < nB * chi) {
        const int rr = idx / chi, kp = idx - (idx / chi) * chi;
        A0[colid[rr] * DS + kp] = v[u];  // V [(t,b)][k'] or U [(s,a)][k']
      }
    }
    stage_r(A1, vside ? 1 : 0, vside ? rj : ri);
    __syncthreads();
  }
  if constexpr (NMAX == 64) {
    // The three small products below run on the FP64 matrix cores as 16 x 16 output tiles, one
    // tile position per wave with both slices (s or t = 0, 1) in it (at most four positions:
    // D <= 32); results stay in registers across the barrier that frees the LDS they overwrite.
    static_assert(NMAX <= 32 || NT >= 256, "one tile position per wave");
    const int wv = tid >> 6, li = tid & 15, lk = (tid & 63) >> 4;
    auto tile_of = [&](int rows, int& ti, int& tj) {
      const int tn = (chi + 15) >> 4;
      ti = wv / tn;
      tj = wv - ti * tn;
      return wv < ((rows + 15) >> 4) * tn;
    };
    cgemm_d4 ar[2], ai[2];
    int ti = 0, tj = 0;
    if (!vside) {
      // Y_s = R_i^(s)H U_s;  T_j^(t) = lambda/sigma sum_s g(s,t) conj(Y_s);  Z_t = sum_s conj(g(s,t)) Y_s
      const bool tw = tile_of(de, ti, tj);
      if (tw) {
  #pragma unroll
        for (int h = 0; h < 2; ++h) {
          auto fa = [&](int k, int a) -> double2 {
            return cconj(A1[h * DM * DS + a * DS + k]);
          };
          auto fb = [&](int a, int kp) -> double2 {
            return A0[(h * ri + a) * DS + kp];
          };
          cgemm_tile(16 * ti, 16 * tj, de, chi, ri, fa, fb, ar[h], ai[h]);
        }
  #pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int k = 16 * ti + lk + 4 * r, kp = 16 * tj + li;
          const double2 y0 = make_double2(ar[0][r], ai[0][r]), y1 = make_double2(ar[1][r], ai[1][r]);
          if (k < de && kp < chi) {
            const double f = lam_old[k] / sig[perm[kp]];
            putT(2, k, kp, cscale(cadd(cmulc(y0, g00), cmulc(y1, g10)), f));
            putT(3, k, kp, cscale(cadd(cmulc(y0, g01), cmulc(y1, g11)), f));
          }
          const double2 z0 = cadd(cmulc(g00, y0), cmulc(g10, y1)), z1 = cadd(cmulc(g01, y0), cmulc(g11, y1));
          ar[0][r] = z0.x;
          ai[0][r] = z0.y;
          ar[1][r] = z1.x;
          ai[1][r] = z1.y;
        }
      }
      __syncthreads();
      if (tw) {
  #pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int k = 16 * ti + lk + 4 * r, kp = 16 * tj + li;
          if (k < de && kp < chi) {
            A0[k * DS + kp] = make_double2(ar[0][r], ai[0][r]);
            A0[DM * DS + k * DS + kp] = make_double2(ar[1][r], ai[1][r]);
          }
        }
      }
      stage_r(A1, 1, rj);
      __syncthreads();
      // V_t[b][k'] = 1/sigma sum_k conj(R_j^(t)[b,k]) lambda_k Z_t[k][k']
      const bool tv = tile_of(rj, ti, tj);
      if (tv) {
  #pragma unroll
        for (int h = 0; h < 2; ++h) {
          auto fa = [&](int b, int k) -> double2 {
            return cscale(cconj(A1[h * DM * DS + b * DS + k]), lam_old[k]);
          };
          auto fb = [&](int k, int kp) -> double2 {
            return A0[h * DM * DS + k * DS + kp];
          };
          cgemm_tile(16 * ti, 16 * tj, rj, chi, de, fa, fb, ar[h], ai[h]);
        }
      }
      __syncthreads();
      if (tv) {
  #pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int b = 16 * ti + lk + 4 * r, kp = 16 * tj + li;
          if (b < rj && kp < chi) {
            const double is = 1.0 / sig[perm[kp]];
            A0[b * DS + kp] = cscale(make_double2(ar[0][r], ai[0][r]), is);
            A0[(rj + b) * DS + kp] = cscale(make_double2(ar[1][r], ai[1][r]), is);
          }
        }
      }
      __syncthreads();
      // T_i^(s) = lambda/sigma sum_t g(s,t) R_j^(t)T V_t
      if (tile_of(de, ti, tj)) {
  #pragma unroll
        for (int h = 0; h < 2; ++h) {
          auto fa = [&](int k, int b) -> double2 {
            return A1[h * DM * DS + b * DS + k];
          };
          auto fb = [&](int b, int kp) -> double2 {
            return A0[(h * rj + b) * DS + kp];
          };
          cgemm_tile(16 * ti, 16 * tj, de, chi, rj, fa, fb, ar[h], ai[h]);
        }
  #pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int k = 16 * ti + lk + 4 * r, kp = 16 * tj + li;
          if (k < de && kp < chi) {
            const double2 x0 = make_double2(ar[0][r], ai[0][r]), x1 = make_double2(ar[1][r], ai[1][r]);
            const double f = lam_old[k] / sig[perm[kp]];
            putT(0, k, kp, cscale(cadd(cmul(g00, x0), cmul(g01, x1)), f));
            putT(1, k, kp, cscale(cadd(cmul(g10, x0), cmul(g11, x1)), f));
          }
        }
      }
    } else {
      // X_t = R_j^(t)T V_t;  T_i^(s) = lambda/sigma sum_t g(s,t) X_t;  P_s = lambda sum_t g(s,t) X_t
      const bool tw = tile_of(de, ti, tj);
      if (tw) {
  #pragma unroll
        for (int h = 0; h < 2; ++h) {
          auto fa = [&](int k, int b) -> double2 {
            return A1[h * DM * DS + b * DS + k];
          };
          auto fb = [&](int b, int kp) -> double2 {
            return A0[(h * rj + b) * DS + kp];
          };
          cgemm_tile(16 * ti, 16 * tj, de, chi, rj, fa, fb, ar[h], ai[h]);
        }
  #pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int k = 16 * ti + lk + 4 * r, kp = 16 * tj + li;
          const double2 x0 = make_double2(ar[0][r], ai[0][r]), x1 = make_double2(ar[1][r], ai[1][r]);
          const double lk_ = k < de ? lam_old[k] : 0.0;
          const double2 p0 = cscale(cadd(cmul(g00, x0), cmul(g01, x1)), lk_);
          const double2 p1 = cscale(cadd(cmul(g10, x0), cmul(g11, x1)), lk_);
          if (k < de && kp < chi) {
            const double is = 1.0 / sig[perm[kp]];
            putT(0, k, kp, cscale(p0, is));
            putT(1, k, kp, cscale(p1, is));
          }
          ar[0][r] = p0.x;
          ai[0][r] = p0.y;
          ar[1][r] = p1.x;
          ai[1][r] = p1.y;
        }
      }
      __syncthreads();
      if (tw) {
  #pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int k = 16 * ti + lk + 4 * r, kp = 16 * tj + li;
          if (k < de && kp < chi) {
            A0[k * DS + kp] = make_double2(ar[0][r], ai[0][r]);
            A0[DM * DS + k * DS + kp] = make_double2(ar[1][r], ai[1][r]);
          }
        }
      }
      stage_r(A1, 0, ri);
      __syncthreads();
      // U_s[a][k'] = 1/sigma sum_k R_i^(s)[a,k] P_s[k][k']
      const bool tu = tile_of(ri, ti, tj);
      if (tu) {
  #pragma unroll
        for (int h = 0; h < 2; ++h) {
          auto fa = [&](int a, int k) -> double2 {
            return A1[h * DM * DS + a * DS + k];
          };
          auto fb = [&](int k, int kp) -> double2 {
            return A0[h * DM * DS + k * DS + kp];
          };
          cgemm_tile(16 * ti, 16 * tj, ri, chi, de, fa, fb, ar[h], ai[h]);
        }
      }
      __syncthreads();
      if (tu) {
  #pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int a = 16 * ti + lk + 4 * r, kp = 16 * tj + li;
          if (a < ri && kp < chi) {
            const double is = 1.0 / sig[perm[kp]];
            A0[a * DS + kp] = cscale(make_double2(ar[0][r], ai[0][r]), is);
            A0[(ri + a) * DS + kp] = cscale(make_double2(ar[1][r], ai[1][r]), is);
          }
        }
      }
      __syncthreads();
      // T_j^(t) = lambda/sigma sum_s g(s,t) R_i^(s)T conj(U_s)
      if (tile_of(de, ti, tj)) {
  #pragma unroll
        for (int h = 0; h < 2; ++h) {
          auto fa = [&](int k, int a) -> double2 {
            return A1[h * DM * DS + a * DS + k];
          };
          auto fb = [&](int a, int kp) -> double2 {
            return cconj(A0[(h * ri + a) * DS + kp]);
          };
          cgemm_tile(16 * ti, 16 * tj, de, chi, ri, fa, fb, ar[h], ai[h]);
        }
  #pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int k = 16 * ti + lk + 4 * r, kp = 16 * tj + li;
          if (k < de && kp < chi) {
            const double2 y0 = make_double2(ar[0][r], ai[0][r]), y1 = make_double2(ar[1][r], ai[1][r]);
            const double f = lam_old[k] / sig[perm[kp]];
            putT(2, k, kp, cscale(cadd(cmul(g00, y0), cmul(g10, y1)), f));
            putT(3, k, kp, cscale(cadd(cmul(g01, y0), cmul(g11, y1)), f));
          }
        }
      }
    }
  } else {
    // D <= 16: every product is one 16 x 16 tile per physical slice, so wave h (h = 0, 1) takes
    // slice h on the matrix cores (one wave takes both when the workgroup has one); the two
    // slices meet in LDS, where every thread combines them for its (k, k') entry.  They meet in A0,
    // once every wave has read what it holds (slices of their own would take 8.7 KB more: five
    // workgroups a CU instead of eight).
    constexpr int NW = NT / 64;
    static_assert(DM <= 16, "one tile per slice");
    const int wv = tid >> 6, li = tid & 15, lk = (tid & 63) >> 4;
    static_assert(DS == 17, "Xs[h][k][k'] is A0[h DM DS + k DS + k']");
    double2 (*const Xs)[16][17] = reinterpret_cast<double2 (*)[16][17]>(A0);
    constexpr int HW = NW == 1 ? 2 : 1;  // slices of a wave in the first product
    cgemm_d4 cr, ci, c1r[HW], c1i[HW];
    auto meet = [&]() {
      __syncthreads();  // A0 has been read
#pragma unroll
      for (int q = 0; q < HW; ++q)
        if (wv + q < 2) {
#pragma unroll
          for (int r = 0; r < 4; ++r) Xs[wv + q][lk + 4 * r][li] = make_double2(c1r[q][r], c1i[q][r]);
        }
      __syncthreads();
    };
    if (!vside) {
      // Y_s = R_i^(s)H U_s;  T_j^(t) = lambda/sigma sum_s g(s,t) conj(Y_s);  Z_t = sum_s conj(g(s,t)) Y_s
#pragma unroll
      for (int q = 0; q < HW; ++q) {
        const int h = wv + q;
        auto fa = [&](int k, int a) -> double2 {
          return cconj(A1[h * DM * DS + a * DS + k]);
        };
        auto fb = [&](int a, int kp) -> double2 {
          return A0[(h * ri + a) * DS + kp];
        };
        if (h < 2) cgemm_tile(0, 0, de, chi, ri, fa, fb, c1r[q], c1i[q]);
      }
      meet();
      for (int idx = tid; idx < 256; idx += NT) {
        const int k = idx >> 4, kp = idx & 15;
        if (k < de && kp < chi) {
          const double2 y0 = Xs[0][k][kp], y1 = Xs[1][k][kp];
          const double f = lam_old[k] / sig[perm[kp]];
          putT(2, k, kp, cscale(cadd(cmulc(y0, g00), cmulc(y1, g10)), f));
          putT(3, k, kp, cscale(cadd(cmulc(y0, g01), cmulc(y1, g11)), f));
          A0[k * DS + kp] = cadd(cmulc(g00, y0), cmulc(g10, y1));
          A0[DM * DS + k * DS + kp] = cadd(cmulc(g01, y0), cmulc(g11, y1));
        }
      }
      stage_r(A1, 1, rj);
      __syncthreads();
      // V_t[b][k'] = 1/sigma sum_k conj(R_j^(t)[b,k]) lambda_k Z_t[k][k'], then
      // X_t = R_j^(t)T V_t (each wave on its own slice: no barrier between the two)
      for (int h = wv; h < 2; h += NW) {
        auto fa = [&](int b, int k) -> double2 {
          return cscale(cconj(A1[h * DM * DS + b * DS + k]), lam_old[k]);
        };
        auto fb = [&](int k, int kp) -> double2 {
          return A0[h * DM * DS + k * DS + kp];
        };
        cgemm_tile(0, 0, rj, chi, de, fa, fb, cr, ci);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double is = li < chi ? 1.0 / sig[perm[li]] : 0.0;
          Xs[h][lk + 4 * r][li] = cscale(make_double2(cr[r], ci[r]), is);
        }
        wave_lds_sync();
        auto fc = [&](int k, int b) -> double2 {
          return A1[h * DM * DS + b * DS + k];
        };
        auto fd = [&](int b, int kp) -> double2 { return Xs[h][b][kp]; };
        cgemm_tile(0, 0, de, chi, rj, fc, fd, cr, ci);
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < 4; ++r) Xs[h][lk + 4 * r][li] = make_double2(cr[r], ci[r]);
      }
      __syncthreads();
      // T_i^(s) = lambda/sigma sum_t g(s,t) X_t
      for (int idx = tid; idx < 256; idx += NT) {
        const int k = idx >> 4, kp = idx & 15;
        if (k < de && kp < chi) {
          const double2 x0 = Xs[0][k][kp], x1 = Xs[1][k][kp];
          const double f = lam_old[k] / sig[perm[kp]];
          putT(0, k, kp, cscale(cadd(cmul(g00, x0), cmul(g01, x1)), f));
          putT(1, k, kp, cscale(cadd(cmul(g10, x0), cmul(g11, x1)), f));
        }
      }
    } else {
      // X_t = R_j^(t)T V_t;  T_i^(s) = lambda/sigma sum_t g(s,t) X_t;  P_s = lambda sum_t g(s,t) X_t
#pragma unroll
      for (int q = 0; q < HW; ++q) {
        const int h = wv + q;
        auto fa = [&](int k, int b) -> double2 {
          return A1[h * DM * DS + b * DS + k];
        };
        auto fb = [&](int b, int kp) -> double2 {
          return A0[(h * rj + b) * DS + kp];
        };
        if (h < 2) cgemm_tile(0, 0, de, chi, rj, fa, fb, c1r[q], c1i[q]);
      }
      meet();
      for (int idx = tid; idx < 256; idx += NT) {
        const int k = idx >> 4, kp = idx & 15;
        if (k < de && kp < chi) {
          const double2 x0 = Xs[0][k][kp], x1 = Xs[1][k][kp];
          const double2 p0 = cscale(cadd(cmul(g00, x0), cmul(g01, x1)), lam_old[k]);
          const double2 p1 = cscale(cadd(cmul(g10, x0), cmul(g11, x1)), lam_old[k]);
          const double is = 1.0 / sig[perm[kp]];
          putT(0, k, kp, cscale(p0, is));
          putT(1, k, kp, cscale(p1, is));
          A0[k * DS + kp] = p0;
          A0[DM * DS + k * DS + kp] = p1;
        }
      }
      stage_r(A1, 0, ri);
      __syncthreads();
      // U_s[a][k'] = 1/sigma sum_k R_i^(s)[a,k] P_s[k][k'], then Y_s = R_i^(s)T conj(U_s)
      for (int h = wv; h < 2; h += NW) {
        auto fa = [&](int a, int k) -> double2 {
          return A1[h * DM * DS + a * DS + k];
        };
        auto fb = [&](int k, int kp) -> double2 {
          return A0[h * DM * DS + k * DS + kp];
        };
        cgemm_tile(0, 0, ri, chi, de, fa, fb, cr, ci);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double is = li < chi ? 1.0 / sig[perm[li]] : 0.0;
          Xs[h][lk + 4 * r][li] = cscale(make_double2(cr[r], ci[r]), is);
        }
        wave_lds_sync();
        auto fc = [&](int k, int a) -> double2 {
          return A1[h * DM * DS + a * DS + k];
        };
        auto fd = [&](int a, int kp) -> double2 { return cconj(Xs[h][a][kp]); };
        cgemm_tile(0, 0, de, chi, ri, fc, fd, cr, ci);
        wave_lds_sync();
#pragma unroll
        for (int r = 0; r < 4; ++r) Xs[h][lk + 4 * r][li] = make_double2(cr[r], ci[r]);
      }
      __syncthreads();
      // T_j^(t) = lambda/sigma sum_s g(s,t) Y_s
      for (int idx = tid; idx < 256; idx += NT) {
        const int k = idx >> 4, kp = idx & 15;
        if (k < de && kp < chi) {
          const double2 y0 = Xs[0][k][kp], y1 = Xs[1][k][kp];
          const double f = lam_old[k] / sig[perm[kp]];
          putT(2, k, kp, cscale(cadd(cmul(g00, y0), cmul(g10, y1)), f));
          putT(3, k, kp, cscale(cadd(cmul(g01, y0), cmul(g11, y1)), f));
        }
      }
    }
  }
  if (BWD && !ACC) {
    // the other set of singular vectors for every triplet above kRecTau, through Theta'
    __syncthreads();
    const int ld = 2 * D;
    double2* Ug = st.bU + (int64_t)slot * ld * ld;
    double2* Vg = st.bV + (int64_t)slot * ld * ld;
    const double2* Th = st.wsb + (int64_t)slot * adj_scratch(D) + (int64_t)32 * D * D;  // [2D][2D], formed above
    const double smax = sig[perm[0]];
    const int mO = trans ? n0 : m0;  // rows of the recovered side
    const int kI = trans ? m0 : n0;  // inner dimension
    // O = Theta' V (have V: U = O / sigma) or O = Theta'^H U (have U: V = O / sigma) on the FP64
    // matrix cores, 16 x 16 output tiles over the waves (lane l holds A[l % 16][l / 16] and
    // B[l / 16][l % 16] and receives D[l / 16 + 4 r][l % 16]); triplets at or below kRecTau are zero
    {
      typedef double d4 __attribute__((ext_vector_type(4)));
      const int l = tid & 63, wv = tid >> 6, li = l & 15, lk = l >> 4;
      const int tn = (nB + 15) >> 4, ntile = ((mO + 15) >> 4) * tn, ks = (kI + 3) >> 2;
      const double2* Jv = trans ? Ug : Vg;  // the Jacobi side, [inner][k]
      for (int tile = wv; tile < ntile; tile += NT / 64) {
        const int ti = tile / tn, tj = tile - (tile / tn) * tn;
        const int i = 16 * ti + li, j = 16 * tj + li;
        d4 cr = {0.0, 0.0, 0.0, 0.0}, ci = {0.0, 0.0, 0.0, 0.0};
        for (int s0 = 0; s0 < ks; s0 += 4) {
          double2 a[4], bb[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int kk = 4 * (s0 + u) + lk;
            a[u] = make_double2(0.0, 0.0);
            bb[u] = make_double2(0.0, 0.0);
            if (i < mO && kk < kI) a[u] = trans ? cconj(Th[kk * ld + i]) : Th[i * ld + kk];
            if (j < nB && kk < kI) bb[u] = Jv[kk * ld + j];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (s0 + u < ks) {
              cr = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].x, bb[u].x, cr, 0, 0, 0);
              cr = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[u].y, bb[u].y, cr, 0, 0, 0);
              ci = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].x, bb[u].y, ci, 0, 0, 0);
              ci = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].y, bb[u].x, ci, 0, 0, 0);
            }
          }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int rr = 16 * ti + lk + 4 * r, k = 16 * tj + li;
          if (rr < mO && k < nB) {
            const double sv = sig[perm[k]];
            (trans ? Vg : Ug)[rr * ld + k] =
                sv > kRecTau * smax ? cscale(make_double2(cr[r], ci[r]), 1.0 / sv) : make_double2(0.0, 0.0);
          }
        }
      }
    }
  }
}

// ------------------------------------------------------------------ K3: re-absorb

template <typename CT, int DM = kMaxD>
__global__ __launch_bounds__(256) void k_reabsorb(DevState st, const int32_t* __restrict__ items, int first,
                                                  int blocks_per_slice) {
  int slot, sp, rb;  // sp = side * 2 + slice
  row_task(st, blockIdx.x, blocks_per_slice, slot, sp, rb);
  const int side = sp >> 1, p = sp & 1;
  const int e = items[first + slot];
  const EdgeInfo& E = st.edges[e];
  const SideInfo& S = E.side[side];
  const int D = st.D;
  const int d1 = S.oth[0] >= 0 ? st.chi[S.oth[0]] : 1;
  const int d2 = S.oth[1] >= 0 ? st.chi[S.oth[1]] : 1;
  const int M = d1 * d2;
  const int row0 = rb * kRowBlock;
  if (row0 >= M) return;
  const int rows = min(kRowBlock, M - row0);
  const SlotMeta meta = st.meta[slot];
  const int de = meta.de_old;
  const int ncol = max(de, meta.chi_new);  // columns that may be non-zero before or after

  __shared__ CT Ts[DM][DM + 1];
  __shared__ CT Gs[kRowBlock][DM + 1];
  CT* gam = reinterpret_cast<CT*>(st.gamma);
  const CT* T = reinterpret_cast<const CT*>(st.tbuf) + rbuf_off(st, slot, side, p);
  const int tid = threadIdx.x;
  for (int idx = tid; idx < de * D; idx += blockDim.x) {
    const int k = idx / D, kp = idx - (idx / D) * D;
    Ts[k][kp] = T[k * D + kp];
  }
  const int64_t base = S.goff + p * S.pstride;
  for (int idx = tid; idx < rows * de; idx += blockDim.x) {
    const int rr = idx / de, k = idx - (idx / de) * de;
    const int m = row0 + rr;
    const int o1 = m / d2, o2 = m - (m / d2) * d2;
    Gs[rr][k] = gam[base + (int64_t)o1 * S.so[0] + (int64_t)o2 * S.so[1] + (int64_t)k * S.sq];
  }
  __syncthreads();
  for (int idx = tid; idx < rows * ncol; idx += blockDim.x) {
    const int rr = idx / ncol, kp = idx - (idx / ncol) * ncol;
    const int m = row0 + rr;
    const int o1 = m / d2, o2 = m - (m / d2) * d2;
    CT out;
    if constexpr (sizeof(CT) == sizeof(float2)) {
      float ax = 0.f, ay = 0.f;
      for (int k = 0; k < de; ++k) {
        const CT gv = Gs[rr][k], tv = Ts[k][kp];
        ax += (float)gv.x * (float)tv.x - (float)gv.y * (float)tv.y;
        ay += (float)gv.x * (float)tv.y + (float)gv.y * (float)tv.x;
      }
      out.x = ax;
      out.y = ay;
    } else {
      double ax = 0.0, ay = 0.0;
      for (int k = 0; k < de; ++k) {
        const CT gv = Gs[rr][k], tv = Ts[k][kp];
        ax += gv.x * tv.x - gv.y * tv.y;
        ay += gv.x * tv.y + gv.y * tv.x;
      }
      out.x = ax;
      out.y = ay;
    }
    gam[base + (int64_t)o1 * S.so[0] + (int64_t)o2 * S.so[1] + (int64_t)kp * S.sq] = out;
  }
}

// ------------------------------------------------------------------ K3 (complex64): re-absorb on the matrix cores

// Gamma'^(p) = Gamma^(p) T^(p) for complex64 storage, as four real products per complex one on
// v_mfma_f32_16x16x4f32.  With that instruction, lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16] and receives D[4 (l / 16) + r][l % 16], r = 0..3.  The lane that holds
// Gamma[m][k] in one orientation (A = Gamma, B = T) holds the same element in the other
// (A = T^T, B = Gamma^T), and likewise for T, so the operand registers do not depend on the
// orientation; it is chosen per site layout so that the 16 lanes sharing an output register
// store 16 consecutive addresses: C = Gamma T when the bond leg is the contiguous one,
// C^T = T^T Gamma^T when the rows are.  Each wave owns TPW tiles of 16 rows and every bond
// column (at most 32); operands go from global memory straight to registers.  STREAM marks the
// site-tensor rows nontemporal (read and written once, past the caches) for states far larger
// than the L2 caches.
template <int TPW, int DMX = kMaxD, bool STREAM = false>
__global__ __launch_bounds__(256) void k_reabsorb_mfma(DevState st, const int32_t* __restrict__ items, int first,
                                                       int blocks_per_slice) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  constexpr int RB = 64 * TPW;  // rows per workgroup
  constexpr int KK = DMX / 4;   // k steps of 4 at the largest bond
  constexpr int NT = DMX / 16;  // column tiles of 16 at the largest bond
  int slot, sp, rb;  // sp = side * 2 + slice
  row_task(st, blockIdx.x, blocks_per_slice, slot, sp, rb);
  const int side = sp >> 1, p = sp & 1;
  const int e = items[first + slot];
  const EdgeInfo& E = st.edges[e];
  const SideInfo& S = E.side[side];
  const int D = st.D;
  const int d1 = S.oth[0] >= 0 ? st.chi[S.oth[0]] : 1;
  const int d2 = S.oth[1] >= 0 ? st.chi[S.oth[1]] : 1;
  const int M = d1 * d2;
  if (rb * RB >= M) return;
  const SlotMeta meta = st.meta[slot];
  const int de = meta.de_old;
  const int ncol = max(de, meta.chi_new);  // columns that may be non-zero before or after
  const int ks = (de + 3) >> 2;              // k steps of 4
  const int nt = (ncol + 15) >> 4;           // column tiles of 16
  float2* gam = reinterpret_cast<float2*>(st.gamma);
  const float2* T = reinterpret_cast<const float2*>(st.tbuf) + rbuf_off(st, slot, side, p);
  // (strides in registers: read through S they would be loaded again after every store)
  const int64_t base = S.goff + p * S.pstride, so0 = S.so[0], so1 = S.so[1], sq = S.sq;
  const int64_t rstride = d2 > 1 ? so1 : so0;
  const bool bond_major = sq == 1 || rstride != 1;  // C = Gamma T (else C^T = T^T Gamma^T)
  const int l = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int li = l & 15, lk = l >> 4;

  // T[4 kk + lk][16 t + li]: the same registers serve as B (first form) or A (second form)
  // (indices past the end are clamped and the entries zeroed afterwards: with a test around each
  // load the loads wait for one another.  Whole steps and tiles past the end load nothing.)
  float tr[KK][NT], ti[KK][NT];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      float2 v = make_float2(0.f, 0.f);
      if (kk < ks && t < nt) v = T[min(4 * kk + lk, de - 1) * D + min(16 * t + li, ncol - 1)];
      tr[kk][t] = v.x;
      ti[kk][t] = v.y;
    }
  auto row_off = [&](int m) -> int64_t {
    const int o1 = m / d2, o2 = m - (m / d2) * d2;
    return base + o1 * so0 + o2 * so1;
  };
  // every tile's rows are loaded before the first product (memory-level parallelism); a tile
  // past the last row loads nothing and is skipped below
  float gr[TPW][KK], gi[TPW][KK];
#pragma unroll
  for (int tile = 0; tile < TPW; ++tile) {
    const int row0 = rb * RB + (wave * TPW + tile) * 16;
    const int64_t ro = row_off(min(row0 + li, M - 1));
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      float2 v = make_float2(0.f, 0.f);
      if (row0 < M && kk < ks) v = ld_c64(&gam[ro + min(4 * kk + lk, de - 1) * sq], STREAM);
      gr[tile][kk] = v.x;
      gi[tile][kk] = v.y;
    }
  }
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const bool kv = 4 * kk + lk < de;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const bool v = kv && 16 * t + li < ncol;
      tr[kk][t] = v ? tr[kk][t] : 0.f;
      ti[kk][t] = v ? ti[kk][t] : 0.f;
    }
#pragma unroll
    for (int tile = 0; tile < TPW; ++tile) {
      const bool v = kv && rb * RB + (wave * TPW + tile) * 16 + li < M;
      gr[tile][kk] = v ? gr[tile][kk] : 0.f;
      gi[tile][kk] = v ? gi[tile][kk] : 0.f;
    }
  }
#pragma unroll
  for (int tile = 0; tile < TPW; ++tile) {
    const int row0 = rb * RB + (wave * TPW + tile) * 16;
    if (row0 >= M) break;
    // three real products per complex one: P1 = Gr Tr, P2 = Gi Ti, P3 = (Gr + Gi)(Tr + Ti);
    // Re C = P1 - P2, Im C = P3 - P1 - P2
    f4 q1[NT], q2[NT], q3[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      q1[t] = (f4){0.f, 0.f, 0.f, 0.f};
      q2[t] = (f4){0.f, 0.f, 0.f, 0.f};
      q3[t] = (f4){0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (kk < ks) {
        const float gs = gr[tile][kk] + gi[tile][kk];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (t < nt) {
            const float ts = tr[kk][t] + ti[kk][t];
            if (bond_major) {  // C[m][k'] = sum_k Gamma[m][k] T[k][k']
              q1[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(gr[tile][kk], tr[kk][t], q1[t], 0, 0, 0);
              q2[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(gi[tile][kk], ti[kk][t], q2[t], 0, 0, 0);
              q3[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(gs, ts, q3[t], 0, 0, 0);
            } else {           // C^T[k'][m] = sum_k T^T[k'][k] Gamma^T[k][m]
              q1[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(tr[kk][t], gr[tile][kk], q1[t], 0, 0, 0);
              q2[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(ti[kk][t], gi[tile][kk], q2[t], 0, 0, 0);
              q3[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(ts, gs, q3[t], 0, 0, 0);
            }
          }
        }
      }
    }
    f4 cr[NT], ci[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      cr[t] = q1[t] - q2[t];
      ci[t] = q3[t] - q1[t] - q2[t];
    }
    // the rows of this tile were read into registers above; write the new rows.  A lane's rows
    // are m0, m0 + 1, ... (first form) or m0 four times (second form): one division, then
    // the other-leg indices (o1, o2) step forward.
    const int m0 = bond_major ? row0 + 4 * lk : row0 + li;
    int o1 = m0 / d2, o2 = m0 - (m0 / d2) * d2;
    int64_t roff[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      roff[r] = base + o1 * so0 + o2 * so1;
      if (bond_major && ++o2 == d2) {
        o2 = 0;
        ++o1;
      }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t < nt) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = bond_major ? m0 + r : m0;
          const int kp = bond_major ? 16 * t + li : 16 * t + 4 * lk + r;
          if (m < M && kp < ncol)
            st_c64(&gam[roff[r] + kp * sq], make_float2(cr[t][r], ci[t][r]), STREAM);
        }
      }
    }
  }
}

// ------------------------------------------------------------------ RX layer

// Gamma_v[0] <- c Gamma_v[0] - i s Gamma_v[1];  Gamma_v[1] <- -i s Gamma_v[0] + c Gamma_v[1]
template <typename CT>
__global__ __launch_bounds__(256) void k_rx(DevState st, int chunk_first, int advance) {
  // the RX layer that opens a recorded step advances the step counter (the readout that closes
  // the step writes history row counter - 1)
  if (advance && blockIdx.x == 0 && threadIdx.x == 0) *st.step_ctr += 1;
  const int64_t ch = st.chunks[chunk_first + blockIdx.x];
  const int v = (int)(ch >> 32);
  const int cidx = (int)(ch & 0xffffffff);
  const VertexInfo& V = st.verts[v];
  const InstParam ip = st.inst[V.inst];
  int64_t ps = 1;
  for (int l = 0; l < V.deg; ++l) ps *= st.D;
  CT* gam = reinterpret_cast<CT*>(st.gamma) + V.goff;
  const int64_t i0 = (int64_t)cidx * 1024;
  const double c = ip.rx_c, s = ip.rx_s;
  for (int64_t i = i0 + threadIdx.x; i < i0 + 1024 && i < ps; i += blockDim.x) {
    const double2 a = to_d2(gam[i]);
    const double2 b = to_d2(gam[i + ps]);
    // -i s b = (s b.y, -s b.x)
    const double2 na = make_double2(c * a.x + s * b.y, c * a.y - s * b.x);
    const double2 nb = make_double2(s * a.y + c * b.x, -s * a.x + c * b.y);
    gam[i] = from_d2<CT>(na);
    gam[i + ps] = from_d2<CT>(nb);
  }
}

// ------------------------------------------------------------------ <Z> readout

// One workgroup of NT threads per qubit.  Bound by the bytes of the tensors when every CU has
// workgroups enough, by the loads one workgroup has in flight when a single graph's few large
// tensors are read (36 of 512 KB at D = 32, 4 MB at D = 64): each thread keeps the elements of UA
// indices of the outermost leg in flight, and above D = 16 the workgroup has 1024 threads.  One
// 127-qubit instance with full bonds: 309 -> 69 us at D = 64, 43 -> 13 us at D = 32, 7.3 -> 4.4 us
// at D = 16; 32 instances at D = 32 137 -> 98 us (mean over 20 steps, the inactive parts unread).
template <typename CT, int DM, int NT>
__global__ __launch_bounds__(NT) void k_expect_z(DevState st, int v_first, int record) {
  constexpr int UA = 8;
  const int v = v_first + blockIdx.x;
  const VertexInfo& V = st.verts[v];
  const int D = st.D;
  __shared__ double lw[kMaxDeg][DM];
  __shared__ double red0[NT / 64], red1[NT / 64];
  const int tid = threadIdx.x;
  for (int idx = tid; idx < kMaxDeg * D; idx += NT) {
    const int l = idx / D, k = idx - (idx / D) * D;
    double w = 1.0;
    if (l < V.deg) {
      const double x = st.lam[(int64_t)V.leg[l] * D + k];
      w = x * x;
    }
    lw[l][k] = w;
  }
  __syncthreads();
  // threads take the inner legs j (their weight computed once, loads coalesced across threads)
  // and loop over the active indices of the outermost leg a; with fewer inner indices than threads
  // the threads form G groups of `inner`, group g taking a = g, g + G, ...  Past the active indices
  // of a leg the tensor is zero: nothing is read there.  (Told by the index, not by a weight of zero: where a
  // tiny lambda squares to zero an infinite element has to end in the status.)
  int inner = 1;
  for (int l = 1; l < V.deg; ++l) inner *= D;
  const int na = V.deg >= 1 ? st.chi[V.leg[0]] : 1;
  const int n1 = V.deg >= 2 ? st.chi[V.leg[1]] : 1, n2 = V.deg == 3 ? st.chi[V.leg[2]] : 1;
  const int ps = inner * (V.deg >= 1 ? D : 1);
  const CT* gam = reinterpret_cast<const CT*>(st.gamma) + V.goff;
  double r0 = 0.0, r1 = 0.0;
  const int G = inner < NT ? NT / inner : 1;
  const int g = inner < NT ? tid / inner : 0;
  if (g < G) {
    for (int j = tid - g * inner; j < inner; j += NT) {
      const int j1 = V.deg == 3 ? j / D : j, j2 = V.deg == 3 ? j - (j / D) * D : 0;
      if (j1 >= n1 || j2 >= n2) continue;
      const double w = lw[1][j1] * lw[2][j2];  // (1 for a missing leg)
      for (int a0 = g; a0 < na; a0 += UA * G) {
        CT x0[UA], x1[UA];
#pragma unroll
        for (int u = 0; u < UA; ++u) {
          const int a = a0 + u * G;
          const int i = (a < na ? a : a0) * inner + j;
          x0[u] = gam[i];
          x1[u] = gam[i + ps];
        }
#pragma unroll
        for (int u = 0; u < UA; ++u) {
          const int a = a0 + u * G;
          if (a < na) {
            const double wa = V.deg >= 1 ? w * lw[0][a] : w;
            r0 += cabs2(to_d2(x0[u])) * wa;
            r1 += cabs2(to_d2(x1[u])) * wa;
          }
        }
      }
    }
  }
  r0 = group_sum_dpp(r0, 64);
  r1 = group_sum_dpp(r1, 64);
  if ((tid & 63) == 0) {
    red0[tid >> 6] = r0;
    red1[tid >> 6] = r1;
  }
  __syncthreads();
  if (tid == 0) {
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) {
      a += red0[w];
      b += red1[w];
    }
    const double zv = (a - b) / (a + b);
    if (!isfinite(zv)) flag_status(st.status, kStatusNonFinite);
    st.z[v] = zv;
    if (record) {
      const int row = *st.step_ctr - 1;  // the step's RX layer has advanced the counter
      if (row >= 0 && row < st.max_steps) st.hist[(int64_t)row * st.NV + v] = zv;
    }
  }
}


// ------------------------------------------------------------------ product state |0...0>

template <typename CT>
__global__ __launch_bounds__(256) void k_fill_zero(void* p, int64_t n) {
  CT* a = reinterpret_cast<CT*>(p);
  const CT zero = from_d2<CT>(make_double2(0.0, 0.0));
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    a[i] = zero;
}

template <typename CT>
__global__ __launch_bounds__(256) void k_reset(DevState st) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  CT* gam = reinterpret_cast<CT*>(st.gamma);
  for (int64_t v = gid; v < st.NV; v += stride) {
    gam[st.verts[v].goff] = from_d2<CT>(make_double2(1.0, 0.0));
    st.z[v] = 1.0;
  }
  for (int64_t i = gid; i < (int64_t)st.NE * st.D; i += stride) st.lam[i] = (i % st.D) == 0 ? 1.0 : 0.0;
  for (int64_t e = gid; e < st.NE; e += stride) st.chi[e] = 1;
  if (gid == 0) {
    *st.step_ctr = 0;
    *st.status = 0;
  }
  if (gid < kStatLines * kStatStride) st.stats[gid] = 0;
}

// ------------------------------------------------------------------ host-side launchers

// complex64 re-absorb: TPW tiles of 16 rows per wave as tuned (8, 4, 2 or 1)
template <int DMX, bool STREAM>
static void launch_reabsorb_mfma(const DevState& st, const int32_t* items, int first, int count, hipStream_t stream) {
  const int tpw = st.tune_rb == 8 ? 8 : st.tune_rb == 4 ? 4 : st.tune_rb == 2 ? 2 : 1;
  const int bps = (st.D * st.D + 64 * tpw - 1) / (64 * tpw);
  const dim3 grid(row_grid(st, count, bps));
  if (tpw == 8)
    hipLaunchKernelGGL((k_reabsorb_mfma<8, DMX, STREAM>), grid, dim3(256), 0, stream, st, items, first, bps);
  else if (tpw == 4)
    hipLaunchKernelGGL((k_reabsorb_mfma<4, DMX, STREAM>), grid, dim3(256), 0, stream, st, items, first, bps);
  else if (tpw == 2)
    hipLaunchKernelGGL((k_reabsorb_mfma<2, DMX, STREAM>), grid, dim3(256), 0, stream, st, items, first, bps);
  else
    hipLaunchKernelGGL((k_reabsorb_mfma<1, DMX, STREAM>), grid, dim3(256), 0, stream, st, items, first, bps);
}

template <typename CT>
static hipError_t launch_set(int which, const DevState& st, const int32_t* items, int first, int count,
                             int blocks_per_slice, hipStream_t stream) {
  if (count <= 0) return hipSuccess;
  constexpr bool kAccumulate = sizeof(CT) == sizeof(double2);  // complex128 path keeps the rotations
  if (st.D > kMaxD) {
    // bond dimensions 33..64: R factors as below at 64 columns, the two-site SVD in k_svd_big
    switch (which) {
      case 1:
        if constexpr (sizeof(CT) == sizeof(float2)) {
          if (st.gram_split) {
            hipLaunchKernelGGL((k_absorb_gram<kMaxDBig, kGramPart>), dim3(count * 4 * kGramSplit), dim3(256), 0, stream, st,
                               items, first);
            hipLaunchKernelGGL((k_absorb_gram<kMaxDBig, kGramEnd>), dim3(count * 4), dim3(256), 0, stream, st, items,
                               first);
          } else {
            hipLaunchKernelGGL(k_absorb_gram<kMaxDBig>, dim3(count * 4), dim3(256), 0, stream, st, items, first);
          }
        } else
          hipLaunchKernelGGL((k_absorb_qr<CT, kMaxDBig, 32>), dim3(count * 4), dim3(256), 0, stream, st, items, first);
        break;
      case 2:
        return launch_svd_big(sizeof(CT) == sizeof(double2), st, items, first, count, stream);
      case 3:
        if constexpr (sizeof(CT) == sizeof(float2)) {
          if (st.stream_gamma)
            launch_reabsorb_mfma<kMaxDBig, true>(st, items, first, count, stream);
          else
            launch_reabsorb_mfma<kMaxDBig, false>(st, items, first, count, stream);
        } else {
          hipLaunchKernelGGL((k_reabsorb<CT, kMaxDBig>), dim3(row_grid(st, count, blocks_per_slice)), dim3(256), 0, stream, st,
                             items, first, blocks_per_slice);
        }
        break;
      default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  switch (which) {
    case 1:
      if constexpr (sizeof(CT) == sizeof(float2)) {
        if (st.D <= 16)
          hipLaunchKernelGGL(k_absorb_gram<16>, dim3(count * 4), dim3(256), 0, stream, st, items, first);
        else
          hipLaunchKernelGGL(k_absorb_gram<32>, dim3(count * 4), dim3(256), 0, stream, st, items, first);
        break;
      }
      if (st.D <= 16) {
        if (st.tune_qr == 8)
          hipLaunchKernelGGL((k_absorb_qr<CT, 16, 8>), dim3(count * 4), dim3(256), 0, stream, st, items, first);
        else
          hipLaunchKernelGGL((k_absorb_qr<CT, 16, 16>), dim3(count * 4), dim3(256), 0, stream, st, items, first);
      } else {
        if (st.tune_qr == 8)
          hipLaunchKernelGGL((k_absorb_qr<CT, 32, 8>), dim3(count * 4), dim3(256), 0, stream, st, items, first);
        else
          hipLaunchKernelGGL((k_absorb_qr<CT, 32, 16>), dim3(count * 4), dim3(256), 0, stream, st, items, first);
      }
      break;
    case 2:
      if (st.D <= 16 && st.tune_svd == 64)
        hipLaunchKernelGGL((k_theta_svd<CT, 64, 32, kAccumulate>), dim3(count), dim3(64), 0, stream, st, items,
                           first);
      else if (st.D <= 16)
        hipLaunchKernelGGL((k_theta_svd<CT, 256, 32, kAccumulate>), dim3(count), dim3(256), 0, stream, st, items,
                           first);
      else
        hipLaunchKernelGGL((k_theta_svd<CT, 256, 64, kAccumulate>), dim3(count), dim3(256), 0, stream, st, items,
                           first);
      break;
    case 3:
      if constexpr (sizeof(CT) == sizeof(float2)) {
        if (st.stream_gamma)
          launch_reabsorb_mfma<kMaxD, true>(st, items, first, count, stream);
        else
          launch_reabsorb_mfma<kMaxD, false>(st, items, first, count, stream);
      } else {
        hipLaunchKernelGGL(k_reabsorb<CT>, dim3(row_grid(st, count, blocks_per_slice)), dim3(256), 0, stream, st, items,
                           first, blocks_per_slice);
      }
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace gpeps

// C++ entry points used by the host driver (gpeps_host.cpp).
namespace gpeps {

hipError_t launch_edge_kernel(int which, bool c128, const DevState& st, const int32_t* items, int first, int count,
                              int blocks_per_slice, hipStream_t stream) {
  return c128 ? launch_set<double2>(which, st, items, first, count, blocks_per_slice, stream)
              : launch_set<float2>(which, st, items, first, count, blocks_per_slice, stream);
}

// The forward SVD update that also keeps every singular triplet and float64 T (reverse sweep).
hipError_t launch_svd_bwd(bool c128, const DevState& st, const int32_t* items, int first, int count,
                          hipStream_t stream) {
  if (count <= 0) return hipSuccess;
  if (c128) {
    if (st.D <= 16 && st.tune_svd == 64)
      hipLaunchKernelGGL((k_theta_svd<double2, 64, 32, true, true>), dim3(count), dim3(64), 0, stream, st, items,
                         first);
    else if (st.D <= 16)
      hipLaunchKernelGGL((k_theta_svd<double2, 256, 32, true, true>), dim3(count), dim3(256), 0, stream, st, items,
                         first);
    else
      hipLaunchKernelGGL((k_theta_svd<double2, 256, 64, true, true>), dim3(count), dim3(256), 0, stream, st, items,
                         first);
  } else {
    if (st.D <= 16 && st.tune_svd == 64)
      hipLaunchKernelGGL((k_theta_svd<float2, 64, 32, false, true>), dim3(count), dim3(64), 0, stream, st, items,
                         first);
    else if (st.D <= 16)
      hipLaunchKernelGGL((k_theta_svd<float2, 256, 32, false, true>), dim3(count), dim3(256), 0, stream, st, items,
                         first);
    else
      hipLaunchKernelGGL((k_theta_svd<float2, 256, 64, false, true>), dim3(count), dim3(256), 0, stream, st, items,
                         first);
  }
  return hipGetLastError();
}

hipError_t launch_rx(bool c128, const DevState& st, int chunk_first, int n_chunks, int advance, hipStream_t stream) {
  if (n_chunks <= 0) return hipSuccess;
  if (c128) hipLaunchKernelGGL(k_rx<double2>, dim3(n_chunks), dim3(256), 0, stream, st, chunk_first, advance);
  else hipLaunchKernelGGL(k_rx<float2>, dim3(n_chunks), dim3(256), 0, stream, st, chunk_first, advance);
  return hipGetLastError();
}

hipError_t launch_expect_z(bool c128, const DevState& st, int v_first, int n_verts, int record, hipStream_t stream) {
  if (n_verts <= 0) return hipSuccess;
  auto go = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(n_verts), dim3(threads), 0, stream, st, v_first, record);
  };
  if (st.D > kMaxD) c128 ? go(k_expect_z<double2, kMaxDBig, 1024>, 1024) : go(k_expect_z<float2, kMaxDBig, 1024>, 1024);
  else if (st.D > 16) c128 ? go(k_expect_z<double2, kMaxD, 1024>, 1024) : go(k_expect_z<float2, kMaxD, 1024>, 1024);
  else c128 ? go(k_expect_z<double2, 16, 256>, 256) : go(k_expect_z<float2, 16, 256>, 256);
  return hipGetLastError();
}

hipError_t launch_reset(bool c128, const DevState& st, int64_t n_gamma, hipStream_t stream) {
  const int64_t blocks64 = (n_gamma + 255) / 256;
  const int blocks = (int)(blocks64 < 65536 ? (blocks64 > 0 ? blocks64 : 1) : 65536);
  if (c128) {
    hipLaunchKernelGGL(k_fill_zero<double2>, dim3(blocks), dim3(256), 0, stream, st.gamma, n_gamma);
    hipLaunchKernelGGL(k_reset<double2>, dim3(256), dim3(256), 0, stream, st);
  } else {
    hipLaunchKernelGGL(k_fill_zero<float2>, dim3(blocks), dim3(256), 0, stream, st.gamma, n_gamma);
    hipLaunchKernelGGL(k_reset<float2>, dim3(256), dim3(256), 0, stream, st);
  }
  return hipGetLastError();
}

}  // namespace gpeps
