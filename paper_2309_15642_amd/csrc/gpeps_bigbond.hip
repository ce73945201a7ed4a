// Two-site update for bond dimensions 33..64 (Results A and "Long time evolution": chi up to
// several hundred in the paper), gfx950.
//
// At D <= 32 the whole two-site matrix Theta' [2 r_i x 2 r_j] (<= 64 x 64 float64 complex, 64 KB)
// is held in LDS by k_theta_svd.  At D = 64 it is 128 x 128 (256 KB), more than the 160 KB of LDS
// of a CU, so this kernel keeps it where it fits:
//   * Theta' is formed once into a per-item HBM scratch (row-major, leading dimension 128) and
//     stays there for the recovery of the second vector set;
//   * the matrix B whose columns are orthogonalised (B = Theta' or Theta'^H, whichever has fewer
//     columns) lives in registers: 512 threads, 8 lanes per column pair, 16 rows per lane, the
//     stationary and the moving column of every pair (128 VGPRs of data per lane);
//   * one-sided (Hestenes) Jacobi with the pairing {c, c ^ m} of the D <= 32 complex64 kernel:
//     blocks of rounds of equal highest bit hb of m; the lanes of a group are spread over the wave
//     and the moving columns pass between its eight groups by one DPP instruction a word, and
//     across waves through an LDS exchange (64 columns, 130 KB); columns carry a scale, so a
//     rotation takes 8 instead of 12 operations per pair of entries (as k_theta_svd at D = 32);
//     between blocks every column goes to its new owner through LDS, the two halves of the groups in
//     turn; into and out of the last block at 128 columns the ids of 64 and more go through the
//     item's HBM scratch;
//   * B is first reduced by Householder QR with column pivoting, B P = Q R (columns in registers,
//     4 lanes each; the pivot column goes through LDS every step), and the Jacobi iteration runs
//     on X = R^H (nB x nB), whose orthogonalised columns are B's right singular vectors with rows
//     permuted by P: the preconditioning of the D <= 32 complex64 kernel, which gives those
//     vectors to high relative accuracy and cuts the sweeps;
//   * after convergence the kept columns, normalised, give one singular-vector set (staged in
//     LDS); the other set is recovered from the stored Theta' as Theta' v / sigma (or
//     Theta'^H u / sigma), accurate to ~2^-52 sigma_0 / sigma for every kept value, and the four
//     re-absorb matrices T follow as in k_theta_svd:
//       T_i^(s)[k,k'] = lambda_k / sigma_k' sum_{t,b} g(s,t) R_j^(t)[b,k] V[(t,b),k'],
//       T_j^(t)[k,k'] = lambda_k / sigma_k' sum_{s,a} g(s,t) conj(U[(s,a),k']) R_i^(s)[a,k].
// A sweep ends the iteration when it rotates nothing, or (complex64 storage) when all its
// rotations had |g|^2 <= 1e-8 al be, as in k_theta_svd; complex128 here has no quiet level.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "gpeps_device.h"
#include "gpeps_internal.h"

namespace gpeps {

namespace {

constexpr int kBT = 512;                 // threads per item
constexpr int kBN = 2 * kMaxDBig;        // 128: largest side of Theta'
constexpr int kBLJ = 8;                  // lanes per column pair
constexpr int kBRPL = kBN / kBLJ;        // 16 rows per lane
constexpr int kBGroups = kBT / kBLJ;     // 64 lane groups (column pairs)
constexpr double kQuietBigC64 = 1e-8;    // (1e-4)^2, as the complex64 path of k_theta_svd

__device__ __forceinline__ int ins_bit(int g, int hb, int bit) {
  return ((g >> hb) << (hb + 1)) | (bit << hb) | (g & ((1 << hb) - 1));
}

}  // namespace

template <typename CT>
__global__ __launch_bounds__(kBT) void k_svd_big(DevState st, const int32_t* __restrict__ items, int first) {
  constexpr bool C64 = sizeof(CT) == sizeof(float2);
  // 130 KB: column exchange, then the kept vectors [k'][row].  With this stride the 8 lane groups of
  // a wave, 2 rows each, cover all LDS banks once.
  __shared__ double2 X[kBGroups][kBN + 2];
  __shared__ double nrmx[kBN];          // tracked squared norms by column id (exchanges)
  __shared__ double sclx[kBN];          // squared scales of the columns, the same way
  __shared__ double sig[kBN];
  __shared__ int perm[kBN];
  __shared__ int colid_sh[kBN];  // original column of each pivot position
  __shared__ double lam_old[kMaxDBig];
  __shared__ double red_w[kBT / 64];
  __shared__ int sh_flag[3][2];
  __shared__ int sh_chi;
  __shared__ double sh_norm, sh_floor;

  const int slot = blockIdx.x;
  const int e = items[first + slot];
  const EdgeInfo& E = st.edges[e];
  const InstParam ip = st.inst[E.inst];
  const int D = st.D;
  const int tid = threadIdx.x;
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
  const double2* Rg = st.rbuf + rbuf_off(st, slot, 0, 0);  // blocks i0, i1, j0, j1, each [D][D]
  double2* Tg = st.big + (int64_t)slot * big_scratch(D);  // Theta' [m0][n0], leading dimension kBN
  double2* Rs = Tg + kBN * kBN;                            // R by pivot position: Rs[pos][row]
  double2* Og = Rs + kBN * kBN;                            // exchange, then the other vector set

  if (tid < kMaxDBig) lam_old[tid] = tid < de ? lam_e[tid] : 0.0;
  if (tid < 6) sh_flag[tid >> 1][tid & 1] = 0;

  __syncthreads();  // lam_old
  // Theta'[(s,a)][(t,b)] = g(s,t) sum_k R_i^(s)[a,k] lambda_k R_j^(t)[b,k]: 16 x 16 tiles on the
  // FP64 matrix cores, the waves taking the tiles in turn, operands from the R factors
  {
    double fro = 0.0;
    const int wv = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
    const int tm = (m0 + 15) >> 4, tn = (n0 + 15) >> 4;
    auto fa = [&](int i, int k) -> double2 {
      const int s = i / ri, a = i - (i / ri) * ri;
      return cscale(Rg[(int64_t)s * D * D + a * D + k], lam_old[k]);
    };
    auto fb = [&](int k, int j) -> double2 {
      const int t = j / rj, b = j - (j / rj) * rj;
      return Rg[(int64_t)(2 + t) * D * D + b * D + k];
    };
    for (int tile = wv; tile < tm * tn; tile += kBT / 64) {
      const int ti = tile / tn, tj = tile - (tile / tn) * tn;
      cgemm_d4 cr, ci;
      cgemm_tile<true>(16 * ti, 16 * tj, m0, n0, de, fa, fb, cr, ci);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * ti + lk + 4 * r, col = 16 * tj + li;
        if (row < m0 && col < n0) {
          const double2 v = cmul(make_double2(cr[r], ci[r]), gate_phase(ip, row / ri, col / rj));
          Tg[row * kBN + col] = v;
          fro += cabs2(v);
        }
      }
    }
    fro = group_sum_dpp(fro, 64);
    if ((tid & 63) == 0) red_w[tid >> 6] = fro;
  }
  __syncthreads();
  if (tid == 0) {
    double f = 0.0;
    for (int w = 0; w < kBT / 64; ++w) f += red_w[w];
    sh_floor = f * st.trunc_rel * st.trunc_rel * 2.220446049250313e-16;
  }

  // B[c][r] = Theta'[r][c] (not trans) or conj(Theta'[c][r]) (trans), from the HBM copy
  auto b_at = [&](int c, int rr) -> double2 {
    return trans ? cconj(Tg[c * kBN + rr]) : Tg[rr * kBN + c];
  };
  __syncthreads();  // sh_floor

  // Householder QR with column pivoting, B P = Q R (only R is kept).  Column c sits in the
  // registers of lanes 4c .. 4c + 3 (rows ql + 4u); pivoting is virtual (colid records the
  // order).  Every step: the pivot comes from the per-wave candidates of the previous step, its
  // owners build the reflector and put it in LDS (zero above row j), every other group applies it
  // to its own column and publishes the next candidate.  Row blocks above row j are skipped (their
  // test is uniform).  The key of a candidate is the squared norm with its 7 lowest mantissa bits
  // replaced by 127 - column (ties within 2^-45 relative go to the lowest column); a zero
  // norm keeps key 0, a column that cannot be chosen has key -1.  Bound by issue and by the LDS reads
  // of the reflector.  With every group rebuilding the reflector and a test per row, 17.0 k cycles a
  // step at 128 columns.
  {
    constexpr int LQ = kBT / kBN;  // 4 lanes per column
    constexpr int RQ = kBN / LQ;   // 32 rows per lane
    __shared__ double2 pcol[kBN];  // the reflector v = x - beta e_j, zero above row j
    __shared__ double sh_tau;      // I - tau v v^H; 0 when the column is zero below row j
    __shared__ double cand[2][kBT / 64];
    __shared__ int posof[kBN];
    const int qc = tid / LQ, ql = tid - (tid / LQ) * LQ, wv = tid >> 6;
    double2 x[RQ];
#pragma unroll
    for (int u = 0; u < RQ; ++u) {
      const int rr = ql + LQ * u;
      x[u] = (qc < nB && rr < mB) ? b_at(qc, rr) : make_double2(0.0, 0.0);
    }
    auto publish = [&](double s2, bool valid, int buf) {
      double key = -1.0;
      if (valid)
        key = s2 > 0.0 ? __longlong_as_double((__double_as_longlong(s2) & ~127ll) | (long long)(127 - qc)) : 0.0;
      const double m = wave_max_uniform(key);
      if ((tid & 63) == 0) cand[buf][wv] = m;
    };
    {
      double s2 = 0.0;
#pragma unroll
      for (int u = 0; u < RQ; ++u) s2 += cabs2(x[u]);
      publish(group_sum_dpp(s2, LQ), qc < nB, 0);
    }
    if (tid < kBN) posof[tid] = -1;
    bool used = false;
    int jP = 0;
    double2 betaP = make_double2(0.0, 0.0);
    __syncthreads();
    int j = 0;
    for (; j < nB; ++j) {
      double best = cand[j & 1][0];
#pragma unroll
      for (int w = 1; w < kBT / 64; ++w) best = fmax(best, cand[j & 1][w]);
      if (!(best > 0.0)) break;  // the remaining columns are zero below row j
      const int P = 127 - (int)(__double_as_longlong(best) & 127ll);
      if (qc == P) {
        double sb = 0.0;
#pragma unroll
        for (int u = 0; u < RQ; ++u)
          if (LQ * u + LQ > j) {
            const int rr = ql + LQ * u;
            pcol[rr] = rr >= j ? x[u] : make_double2(0.0, 0.0);
            if (rr > j) sb += cabs2(x[u]);
          }
        sb = group_sum_dpp(sb, LQ);
        wave_lds_sync();
        const double2 alpha = pcol[j];
        used = true;
        jP = j;
        betaP = alpha;
        double tau = 0.0;
        if (sb > 0.0) {
          // beta = -phase(x_j) ||x||
          const double aa2 = cabs2(alpha);
          const double nu2 = aa2 + sb;
          const double nu = nu2 * rsq_nr(nu2);
          const double2 ph = aa2 > 0.0 ? cscale(alpha, rsq_nr(aa2)) : make_double2(1.0, 0.0);
          betaP = cscale(ph, -nu);
          const double2 v0 = csub(alpha, betaP);
          tau = 2.0 * rcp_nr(cabs2(v0) + sb);
          wave_lds_sync();
          if (ql == 0) pcol[j] = v0;
        }
        if (ql == 0) {
          sh_tau = tau;
          posof[P] = j;
        }
      }
      __syncthreads();
      double s2 = 0.0;
      if (!used && qc < nB) {
        const double tau = sh_tau;
        double2 f = make_double2(0.0, 0.0);
        if (tau > 0.0) {
          double wr = 0.0, wi = 0.0;
#pragma unroll
          for (int u = 0; u < RQ; ++u)
            if (LQ * u + LQ > j) {
              const double2 v = pcol[ql + LQ * u];
              wr = fma(v.y, x[u].y, fma(v.x, x[u].x, wr));
              wi = fma(-v.y, x[u].x, fma(v.x, x[u].y, wi));
            }
          group_sum2_dpp(wr, wi, LQ);
          f = make_double2(wr * tau, wi * tau);
        }
#pragma unroll
        for (int u = 0; u < RQ; ++u)
          if (LQ * u + LQ > j) {
            const int rr = ql + LQ * u;
            const double2 v = pcol[rr];
            x[u].x = fma(-v.x, f.x, fma(v.y, f.y, x[u].x));
            x[u].y = fma(-v.x, f.y, fma(-v.y, f.x, x[u].y));
            if (rr > j) s2 += cabs2(x[u]);
          }
      }
      publish(group_sum_dpp(s2, LQ), !used && qc < nB, (j + 1) & 1);
      __syncthreads();
    }
    // R's pivot columns: beta on the diagonal, zeros below; never-pivoted (zero below row j)
    // columns follow in ascending order
    if (used && qc < nB) {
#pragma unroll
      for (int u = 0; u < RQ; ++u) {
        const int rr = ql + LQ * u;
        if (rr == jP) x[u] = betaP;
        else if (rr > jP) x[u] = make_double2(0.0, 0.0);
      }
    }
    if (tid == 0)
      for (int c = 0, k = j; c < nB; ++c)
        if (posof[c] < 0) posof[c] = k++;
    __syncthreads();
    if (qc < nB) {
      const int pos = posof[qc];
#pragma unroll
      for (int u = 0; u < RQ; ++u) {
        const int rr = ql + LQ * u;
        if (rr < nB) Rs[pos * kBN + rr] = rr < mB ? x[u] : make_double2(0.0, 0.0);
      }
    }
    if (tid < nB) perm[posof[tid]] = tid;  // perm[pos] = original column (reused below for sorting)
    __syncthreads();
    if (tid < nB) colid_sh[tid] = perm[tid];
    __syncthreads();
  }
  // the Jacobi matrix X = R^H (nB x nB): X[c][r] = conj(R(c, r)) = conj(Rs[r][c])
  auto x_at = [&](int c, int rr) -> double2 { return cconj(Rs[rr * kBN + c]); };
  // lane group and lane of the group: group index inside the wave (blk, low), blk in lane bits 2 and
  // 3, low in lane bit 1; the lanes of a group are lane bits 0, 4 and 5
  const int wl = tid & 63;
  const int pair_id = (tid >> 6) * 8 + ((((wl >> 2) & 3) << 1) | ((wl >> 1) & 1));
  const int lane = (wl & 1) + 2 * (wl >> 4);
  const double own = ((wl >> 4) >> 1) == ((wl & 3) >> 1) ? 1.0 : 0.0;  // the two groups of a block apart
  auto xrow = [&](int u) { return lane + kBLJ * u; };
  // sums over the lanes of a group, against ones on v_mfma_f64_4x4x4 (lane l supplies A[l % 4][l / 16]
  // and B[l / 16][l % 4] of block (l / 4) % 4 and receives D[l / 16][l % 4])
  auto total2 = [&](double& a, double& b) {
    a = own * __builtin_amdgcn_mfma_f64_4x4x4f64(a, 1.0, 0.0, 0, 0, 0);
    b = own * __builtin_amdgcn_mfma_f64_4x4x4f64(b, 1.0, 0.0, 0, 0, 0);
    a = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, a, 0.0, 0, 0, 0);
    b = __builtin_amdgcn_mfma_f64_4x4x4f64(1.0, b, 0.0, 0, 0, 0);
  };
  int K = 1;
  while ((1 << K) < nB) ++K;
  const bool gact = pair_id < (1 << (K - 1));
  const double tol2 = (2.220446049250313e-16 * (double)nB) * (2.220446049250313e-16 * (double)nB);
  // The iteration, the sort and the kept columns, with RB row blocks of kBLJ rows: a matrix of fewer rows leaves
  // the others out, and the waves whose groups are all inactive take part in the barriers only.
  auto iterate = [&](auto row_blocks) {
    constexpr int RB = decltype(row_blocks)::value;
    const bool wact = RB == kBRPL || (__builtin_amdgcn_readfirstlane(tid) >> 6) * 8 < (1 << (K - 1));
    double2 xs[RB], xm[RB];  // stationary and moving column of the group
    double ns = 0.0, nm = 0.0;  // their tracked squared norms
    double ps = 1.0, pm = 1.0;  // their squared scales: the column is sqrt(ps) xs
    int cs_id = ins_bit(pair_id, 0, 0), cm_id = ins_bit(pair_id, 0, 1);
    // both scales folded into the columns, their squared norms to ns, nm
    auto fold = [&]() {
      const double ds = ps * rsq_nr(ps), dm = pm * rsq_nr(pm);
      ns = 0.0;
      nm = 0.0;
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        xs[u] = cscale(xs[u], ds);
        xm[u] = cscale(xm[u], dm);
        ns += cabs2(xs[u]);
        nm += cabs2(xm[u]);
      }
      ps = 1.0;
      pm = 1.0;
      total2(ns, nm);
    };
    // initial assignment (block hb = 0): group g holds columns 2g and 2g + 1
#pragma unroll
    for (int u = 0; u < RB; ++u) {
      const int rr = xrow(u);
      xs[u] = (gact && cs_id < nB && rr < nB) ? x_at(cs_id, rr) : make_double2(0.0, 0.0);
      xm[u] = (gact && cm_id < nB && rr < nB) ? x_at(cm_id, rr) : make_double2(0.0, 0.0);
    }
    const double floor2 = sh_floor * sh_floor;

    // Every column to its owner under block hb.  Within the blocks hb < 6 the ids under 64 stay with
    // the first half of the groups and the others with the second half, so the halves take turns with
    // the LDS buffer; into and out of block 6 (two of the seven times a sweep at 128 columns) the ids
    // of 64 and more go through the item's HBM scratch.  All through the two buffers at once: 26 k
    // cycles a time.
    auto redistribute = [&](int hb, int from) {
      const bool turns = hb < 6 && from < 6;
      auto put = [&](const double2 (&x)[RB], int c, double n2, double p2) {
        if (!gact || c >= nB) return;
        double2* dst = turns ? &X[c & (kBGroups - 1)][0] : c < kBGroups ? &X[c][0] : Og + (int64_t)(c - kBGroups) * kBN;
#pragma unroll
        for (int u = 0; u < RB; ++u) dst[xrow(u)] = x[u];
        if (lane == 0) {
          nrmx[c] = n2;
          sclx[c] = p2;
        }
      };
      auto get = [&](double2 (&x)[RB], int c, double& n2, double& p2) {
        const bool ok = gact && c < nB;
        const double2* src = turns ? &X[c & (kBGroups - 1)][0]
                                   : c < kBGroups ? &X[c][0] : Og + (int64_t)(c - kBGroups) * kBN;
#pragma unroll
        for (int u = 0; u < RB; ++u) {
          const double2 t = src[xrow(u)];
          x[u] = ok ? t : make_double2(0.0, 0.0);
        }
        n2 = ok ? nrmx[c] : 0.0;
        p2 = ok ? sclx[c] : 1.0;
      };
      const bool second = pair_id >= kBGroups / 2;
      const int n_turns = turns && nB > kBGroups ? 2 : 1;
      for (int turn = 0; turn < n_turns; ++turn) {
        const bool mine = !turns || second == (turn == 1);
        if (mine) {
          put(xs, cs_id, ns, ps);
          put(xm, cm_id, nm, pm);
        }
        __syncthreads();
        if (mine) {
          cs_id = ins_bit(pair_id, hb, 0);
          cm_id = ins_bit(pair_id, hb, 1);
          get(xs, cs_id, ns, ps);
          get(xm, cm_id, nm, pm);
        }
        __syncthreads();
      }
    };

    bool rot = false, big = false;
    int sweep = 0;
    bool converged = nB < 2;
    for (; sweep < st.max_sweeps && !converged; ++sweep) {
      for (int hb = 0; hb < K; ++hb) {
        if (hb == 0) fold();
        const int nt = 1 << hb;
        // rotation of the pair (stationary xs, moving xm) by tan theta e^{i phi} = g F,
        // F = sign(d) / (h x), x = cos^2 theta; branch-free: a pair that is not rotated takes F = 0 and
        // x = 1, which leaves both columns and norms bit for bit
        auto round = [&]() {
          double gr, gi;
          dot_rows<RB>(xs, xm, gr, gi);
          total2(gr, gi);
          const double al = ns, be = nm;
          const double g2 = (gr * gr + gi * gi) * (ps * pm);
          const double ab = al * be;
          // the columns of inactive groups and of ids past nB are exactly zero: g = 0
          const bool ok = (g2 > tol2 * ab) & (g2 > floor2);
          const double d = be - al;
          const double h2 = fmax(d * d + 4.0 * g2, 1e-300);
          const double rh = C64 ? rsq_nr1(h2) : rsq_nr(h2);  // 1 / h
          const double x = 0.5 + 0.5 * fabs(d) * rh;
          const double rx = C64 ? rcp_nr1(x) : rcp_nr(x);    // 1 / x
          const double F = ok ? copysign(rh, d) * rx : 0.0;
          const double xx = ok ? x : 1.0;
          const double tg = g2 * F;  // tan theta |g|
          const double fm = F * pm, fs = F * ps;
          const double2 tm = make_double2(gr * fm, gi * fm), ts = make_double2(gr * fs, gi * fs);
#pragma unroll
          for (int u = 0; u < RB; ++u) {
            const double2 a = xs[u], b = xm[u];
            xs[u].x = fma(-tm.x, b.x, fma(-tm.y, b.y, a.x));
            xs[u].y = fma(-tm.x, b.y, fma(tm.y, b.x, a.y));
            xm[u].x = fma(ts.x, a.x, fma(-ts.y, a.y, b.x));
            xm[u].y = fma(ts.x, a.y, fma(ts.y, a.x, b.y));
          }
          ps *= xx;
          pm *= xx;
          ns = al - tg;
          nm = be + tg;
          rot = rot || ok;
          big = big || (ok && g2 > kQuietBigC64 * ab);
        };
        auto move = [&](auto perm) {  // the moving column, its norm and scale, through a lane permutation
#pragma unroll
          for (int u = 0; u < RB; ++u) xm[u] = make_double2(perm(xm[u].x), perm(xm[u].y));
          nm = perm(nm);
          pm = perm(pm);
        };
        if (nt < 8) {
          // fewer rounds than groups of a wave: group ^ 2^b, b the Gray-code bit
          for (int t = 0; wact && t < nt; ++t) {
            round();
            if (t + 1 < nt) {
              if (__builtin_ctz(t + 1) == 0) move([](double v) { return dpp_d<0x4E>(v); });  // low: lane ^ 2
              else move([](double v) { return lane_xor<4>(v); });                             // blk ^ 1
            }
          }
          cm_id = ins_bit(pair_id ^ ((nt - 1) ^ ((nt - 1) >> 1)), hb, 1);
        } else {
          int T = 0;
          for (;; ++T) {
            // blk turns once more than it has to, so that every trip is the same straight line (a
            // condition on the last one costs copies and spills of the whole column) and the columns
            // end where they began
#pragma unroll 1
            for (int sb = 0; wact && sb < 4; ++sb) {
              round();
              move([](double v) { return dpp_d<0x4E>(v); });  // low ^ 1
              round();
              move([](double v) { return dpp_d<0x124>(v); });  // blk - 1 to blk
            }
            if (8 * (T + 1) >= nt) break;
            // to the wave whose index differs in the next Gray-code bit, same group inside the wave
#pragma unroll
            for (int u = 0; u < RB; ++u) X[pair_id][xrow(u)] = xm[u];
            if (lane == 0) {
              nrmx[pair_id] = nm;
              sclx[pair_id] = pm;
            }
            __syncthreads();
            const int src = pair_id ^ (8 << __builtin_ctz(T + 1));
#pragma unroll
            for (int u = 0; u < RB; ++u) xm[u] = X[src][xrow(u)];
            nm = nrmx[src];
            pm = sclx[src];
            __syncthreads();
          }
          cm_id = ins_bit(pair_id ^ ((T ^ (T >> 1)) << 3), hb, 1);
        }
        if (hb + 1 == K) {
          if (rot && lane == 0) sh_flag[sweep % 3][0] = 1;
          if (big && lane == 0) sh_flag[sweep % 3][1] = 1;
          if (tid < 2) sh_flag[(sweep + 1) % 3][tid] = 0;
          rot = false;
          big = false;
        }
        if (hb + 1 < K) redistribute(hb + 1, hb);
      }
      __syncthreads();
      converged = (sh_flag[sweep % 3][0] == 0) || (C64 && sh_flag[sweep % 3][1] == 0);
      if (!converged) redistribute(0, K - 1);
    }
    fold();
    if (tid == 0) count_svd(st, sweep, converged);

    // singular values (norms of the held columns), stable descending order, truncation
    const double s_s = sqrt(ns), s_m = sqrt(nm);
    if (lane == 0 && gact) {
      if (cs_id < nB) sig[cs_id] = s_s;
      if (cm_id < nB) sig[cm_id] = s_m;
    }
    __syncthreads();
    for (int c = tid; c < nB; c += kBT) perm[falling_rank(sig, nB, c)] = c;
    __syncthreads();
    if (tid == 0) {
      const double smax = sig[perm[0]];
      int keep = 0;
      for (int d2 = 0; d2 < nB; ++d2) keep += sig[d2] > st.trunc_rel * smax;
      int chi = keep < D ? keep : D;
      if (chi < 1) chi = 1;
      double nr = 0.0;
      for (int k = 0; k < chi; ++k) nr += sig[perm[k]] * sig[perm[k]];
      nr = sqrt(nr);
      if (!(smax > 0.0)) flag_status(st.status, kStatusZeroTheta);
      if (!isfinite(nr)) flag_status(st.status, kStatusNonFinite);
      sh_chi = chi;
      sh_norm = nr;
      st.meta[slot].de_old = de;
      st.meta[slot].chi_new = chi;
      st.chi[e] = chi;
    }
    __syncthreads();
    const int chi = sh_chi;
    for (int k = tid; k < D; k += kBT) lam_e[k] = k < chi ? sig[perm[k]] / sh_norm : 0.0;

    // kept columns of X, normalised: B's right singular vectors with rows permuted by the pivoting,
    // X[k'][colid[r]] = x[r] / sigma (rows < nB)
    auto stage = [&](const double2 (&x)[RB], int c, double sv) {
      if (!gact || c >= nB) return;
      const int rank = falling_rank(sig, nB, c);
      if (rank >= chi) return;
      const double inv = sv > 0.0 ? 1.0 / sv : 0.0;
#pragma unroll
      for (int u = 0; u < RB; ++u) {
        const int rr = xrow(u);
        if (rr < nB) X[rank][colid_sh[rr]] = cscale(x[u], inv);
      }
    };
    stage(xs, cs_id, sig[cs_id < nB ? cs_id : 0]);
    stage(xm, cm_id, sig[cm_id < nB ? cm_id : 0]);
    __syncthreads();
  };
  if (nB <= 2 * kBLJ) iterate(std::integral_constant<int, 2>());
  else if (nB <= 4 * kBLJ) iterate(std::integral_constant<int, 4>());
  else iterate(std::integral_constant<int, kBRPL>());
  const int chi = sh_chi;

  // B's right singular vectors are V of Theta' (B = Theta') or U of Theta' (B = Theta'^H); the
  // other set from the stored Theta': U = Theta' V / sigma or V = Theta'^H U / sigma, into
  // Og[row][k'] (leading dimension kMaxDBig)
  const int mO = trans ? n0 : m0;
  {
    const int wv = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
    const int tm = (mO + 15) >> 4, tn = (chi + 15) >> 4;
    auto fa = [&](int i, int q) -> double2 {
      return trans ? cconj(Tg[q * kBN + i]) : Tg[i * kBN + q];
    };
    auto fb = [&](int q, int j) -> double2 {
      return X[j][q];
    };
    for (int tile = wv; tile < tm * tn; tile += kBT / 64) {
      const int ti = tile / tn, tj = tile - (tile / tn) * tn;
      cgemm_d4 cr, ci;
      cgemm_tile<true>(16 * ti, 16 * tj, mO, chi, nB, fa, fb, cr, ci);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int rr = 16 * ti + lk + 4 * r, kp = 16 * tj + li;
        if (rr < mO && kp < chi) {
          const double sv = sig[perm[kp]];
          Og[rr * kMaxDBig + kp] = sv > 0.0 ? cscale(make_double2(cr[r], ci[r]), 1.0 / sv) : make_double2(0.0, 0.0);
        }
      }
    }
  }
  __syncthreads();
  // U[(s,a)][k'] and V[(t,b)][k'] wherever they are
  // (said to be global, or the choice becomes a flat load, which waits for LDS and memory alike)
  typedef double d2 __attribute__((ext_vector_type(2)));
  const __attribute__((address_space(1))) d2* const Om = (const __attribute__((address_space(1))) d2*)Og;
  auto from_x = [&](int row, int kp) -> double2 { return X[kp][row]; };
  auto from_o = [&](int row, int kp) -> double2 {
    const d2 v = Om[row * kMaxDBig + kp];
    return make_double2(v.x, v.y);
  };
  auto Uv = [&](int row, int kp) -> double2 { return trans ? from_x(row, kp) : from_o(row, kp); };
  auto Vv = [&](int row, int kp) -> double2 { return trans ? from_o(row, kp) : from_x(row, kp); };

  CT* T = reinterpret_cast<CT*>(st.tbuf);
  for (int idx = tid; idx < 4 * de * (D - chi); idx += kBT) {
    const int w = idx / (de * (D - chi));
    const int rem = idx - w * de * (D - chi);
    const int k = rem / (D - chi), kp = chi + rem - (rem / (D - chi)) * (D - chi);
    T[rbuf_off(st, slot, w >> 1, w & 1) + k * D + kp] = from_d2<CT>(make_double2(0.0, 0.0));
  }
  const double2 g00 = gate_phase(ip, 0, 0), g01 = gate_phase(ip, 0, 1);
  const double2 g10 = gate_phase(ip, 1, 0), g11 = gate_phase(ip, 1, 1);
  const double2* RI0 = Rg;
  const double2* RI1 = Rg + (int64_t)D * D;
  const double2* RJ0 = Rg + (int64_t)2 * D * D;
  const double2* RJ1 = Rg + (int64_t)3 * D * D;
  // x_t[k][k'] = sum_b R_j^(t)[b][k] V[(t,b)][k'], y_s[k][k'] = sum_a R_i^(s)[a][k] conj(U[(s,a)][k']):
  // four products per 16 x 16 tile of (k, k'), on the matrix cores
  {
    const int wv = tid >> 6, l = tid & 63, li = l & 15, lk = l >> 4;
    const int tm = (de + 15) >> 4, tn = (chi + 15) >> 4;
    for (int tile = wv; tile < tm * tn; tile += kBT / 64) {
      const int ti = tile / tn, tj = tile - (tile / tn) * tn;
      cgemm_d4 xr[2], xi[2], yr[2], yi[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const double2* RJ = h ? RJ1 : RJ0;
        const double2* RI = h ? RI1 : RI0;
        auto fjx = [&](int k, int b) -> double2 {
          return RJ[b * D + k];
        };
        auto fjv = [&](int b, int kp) -> double2 {
          return Vv(h * rj + b, kp);
        };
        auto fix = [&](int k, int a) -> double2 {
          return RI[a * D + k];
        };
        auto fiu = [&](int a, int kp) -> double2 {
          return cconj(Uv(h * ri + a, kp));
        };
        cgemm_tile<true>(16 * ti, 16 * tj, de, chi, rj, fjx, fjv, xr[h], xi[h]);
        cgemm_tile<true>(16 * ti, 16 * tj, de, chi, ri, fix, fiu, yr[h], yi[h]);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = 16 * ti + lk + 4 * r, kp = 16 * tj + li;
        if (k < de && kp < chi) {
          const double2 x0 = make_double2(xr[0][r], xi[0][r]), x1 = make_double2(xr[1][r], xi[1][r]);
          const double2 y0 = make_double2(yr[0][r], yi[0][r]), y1 = make_double2(yr[1][r], yi[1][r]);
          const double f = lam_old[k] / sig[perm[kp]];
          T[rbuf_off(st, slot, 0, 0) + k * D + kp] = from_d2<CT>(cscale(cadd(cmul(g00, x0), cmul(g01, x1)), f));
          T[rbuf_off(st, slot, 0, 1) + k * D + kp] = from_d2<CT>(cscale(cadd(cmul(g10, x0), cmul(g11, x1)), f));
          T[rbuf_off(st, slot, 1, 0) + k * D + kp] = from_d2<CT>(cscale(cadd(cmul(g00, y0), cmul(g10, y1)), f));
          T[rbuf_off(st, slot, 1, 1) + k * D + kp] = from_d2<CT>(cscale(cadd(cmul(g01, y0), cmul(g11, y1)), f));
        }
      }
    }
  }
}

hipError_t launch_svd_big(bool c128, const DevState& st, const int32_t* items, int first, int count,
                          hipStream_t stream) {
  if (count <= 0) return hipSuccess;
  if (st.D > kMaxDBig || !st.big) return hipErrorInvalidValue;
  if (c128) hipLaunchKernelGGL(k_svd_big<double2>, dim3(count), dim3(kBT), 0, stream, st, items, first);
  else hipLaunchKernelGGL(k_svd_big<float2>, dim3(count), dim3(kBT), 0, stream, st, items, first);
  return hipGetLastError();
}

}  // namespace gpeps
