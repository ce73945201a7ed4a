// Adjoint (reverse sweep) of the graph-PEPS simple update for gfx950.
//
// Loss: L = sum_v c_v <Z_v> of the state after the last recorded Trotter step
// (the mean magnetisation of Fig. 2a when c_v = 1/m).  The forward pass stores the
// state at the start of every step (k_checkpoint).  The reverse sweep restores a
// step's checkpoint, recomputes the step while saving the state before each colour
// class, and then reverses the classes in descending order and the RX layer.
//
// One gate, as the forward kernels compute it (per end sigma and physical slice p):
//   A^(p) = Gamma^(p) * w            (w: product of the other legs' lambdas, per row)
//   R^(p): R^H R = A^H A             (Householder, R only)
//   Theta' = [g(s,t) R_i^(s) diag(lambda) R_j^(t)T]_(s,t) = U S V^H, keep chi
//   T_i^(s) = diag(lambda) sum_t g(s,t) R_j^(t)T V_t S^-1,  T_j^(t) = diag(lambda) sum_s g(s,t) R_i^(s)T conj(U_s) S^-1
//   Gamma'^(p) = Gamma^(p) T^(p),  lambda' = S_chi / ||S_chi||
// and its reverse:
//   k_adj_tbar : T-bar = Gamma^H Gamma'-bar                      (row reduction)
//   k_adj_small: T adjoints -> U-bar, V-bar, S-bar, R-bar, lambda-bar, theta_J-bar;
//                complex SVD backward of Theta' (symmetric gauge term, Lorentzian
//                F_kl = d/(d^2 + 1e-12)/(s_k + s_l), d = s_l - s_k in units of s_0);
//                Theta' backward; QR backward
//   k_adj_rows : Gamma-bar = Gamma'-bar T^H + A-bar * w, and lambda-bar of the other legs
// QR backward.  The function of R above is unchanged by R -> W R for any unitary W
// (the singular values are unchanged and V -> conj(W) V cancels in R^T V), so
// R-bar = 2 R G-bar with G-bar Hermitian, and A-bar = 2 A G-bar = A Y, Y = R^-1 R-bar.
// Y is taken from the regularised normal equations (R^H R + delta I) Y = R^H R-bar
// (Gauss-Jordan in LDS, delta = 1e-13 * max diag(R^H R)), then made Hermitian; no Q and no raw
// R^-1 is needed, so rank-deficient slices (frequent at early steps) stay finite.
// When a slice was not reduced (M <= D_e, R = A) A-bar = R-bar directly.
// Complex adjoints follow x-bar = dL/dRe x + i dL/dIm x.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "gpeps_device.h"
#include "gpeps_internal.h"

namespace gpeps {

constexpr double kEpsF = 1e-12;  // Lorentzian broadening of F (singular-value differences, units of s_0)

__device__ __forceinline__ double2 gate_dphase(const InstParam& ip, int s, int t) {
  // d g / d theta_J = -(i/2) z_s z_t g
  const double2 g = gate_phase(ip, s, t);
  const double zz = (s == t) ? 1.0 : -1.0;
  return make_double2(0.5 * zz * g.y, -0.5 * zz * g.x);
}

// block-wide sum of a double (NT threads, result returned to every thread)
template <int NT>
__device__ __forceinline__ double block_sum(double v, double* red) {
  const int tid = threadIdx.x;
  red[tid] = v;
  __syncthreads();
  for (int off = NT / 2; off > 0; off >>= 1) {
    if (tid < off) red[tid] += red[tid + off];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// ------------------------------------------------------------------ checkpoints

// Copy n32 32-bit words from src to dst + (*step_ctr) * slot_words (the history row of this step).
__global__ __launch_bounds__(256) void k_checkpoint(const uint32_t* __restrict__ src, uint32_t* dst,
                                                   int64_t n32, int64_t slot_words, const int32_t* step_ctr,
                                                   int max_steps) {
  const int slot = *step_ctr;
  if (slot >= max_steps) return;
  uint32_t* d = dst + (int64_t)slot * slot_words;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n32; i += (int64_t)gridDim.x * blockDim.x)
    d[i] = src[i];
}

__global__ __launch_bounds__(256) void k_fill_d(double* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.0;
}

// ------------------------------------------------------------------ magnetisation loss

// Mean <Z> over the qubits of every instance from history row `row` (Fig. 2a's magnetisation):
// one workgroup per instance, fixed summation order.
__global__ __launch_bounds__(256) void k_mean_z(DevState st, int row) {
  __shared__ double red[256];
  const int k = blockIdx.x;
  const int vb = st.inst_vb[k], ve = st.inst_vb[k + 1];
  const double* z = st.hist + (int64_t)row * st.NV;
  double acc = 0.0;
  for (int v = vb + (int)threadIdx.x; v < ve; v += 256) acc += z[v];
  const double tot = block_sum<256>(acc, red);
  if (threadIdx.x == 0) st.mean[k] = ve > vb ? tot / (double)(ve - vb) : 0.0;
}

// Seed of the mean-<Z> loss L = sum_k dldm[k] m_k: dL/d<Z_v> = dldm[k] / n_k for v in instance k.
__global__ __launch_bounds__(256) void k_seed_mean(DevState st) {
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v >= st.NV) return;
  const int k = st.verts[v].inst;
  const int n = st.inst_vb[k + 1] - st.inst_vb[k];
  const_cast<double*>(st.dldz)[v] = st.dldm[k] / (double)n;
}

// ------------------------------------------------------------------ readout adjoint (seed)

// z_v = (rho00 - rho11)/(rho00 + rho11), rho_ss = sum_x |Gamma[s,x]|^2 W(x), W = prod_l lambda_l[x_l]^2.
template <typename CT>
__global__ __launch_bounds__(1024) void k_adj_readout(DevState st) {
  constexpr int NT = 1024;  // one large tensor per workgroup: bound by the loads it has in flight
  const int v = blockIdx.x;
  const VertexInfo& V = st.verts[v];
  const int D = st.D, deg = V.deg;
  __shared__ double lw[kMaxDeg][kMaxD];
  __shared__ double acc[kMaxDeg][kMaxD];
  __shared__ double red0[NT / 64], red1[NT / 64];
  const int tid = threadIdx.x;
  for (int idx = tid; idx < kMaxDeg * D; idx += NT) {
    const int l = idx / D, k = idx - (idx / D) * D;
    double w = 1.0;
    if (l < deg) {
      const double x = st.lam[(int64_t)V.leg[l] * D + k];
      w = x * x;
    }
    lw[l][k] = w;
  }
  __syncthreads();
  int ps = 1;
  for (int l = 0; l < deg; ++l) ps *= D;
  const int s0 = deg == 3 ? D * D : deg == 2 ? D : 1, s1 = deg == 3 ? D : 1;  // strides of legs 0 and 1
  auto weight = [&](int i) {
    double w = 1.0;
    if (deg >= 1) w = lw[0][i / s0];
    const int r = i - (i / s0) * s0;
    if (deg >= 2) w *= lw[1][r / s1];
    if (deg >= 3) w *= lw[2][r - (r / s1) * s1];
    return w;
  };
  const CT* gam = reinterpret_cast<const CT*>(st.gamma) + V.goff;
  double r0 = 0.0, r1 = 0.0;
#pragma unroll 4
  for (int i = tid; i < ps; i += NT) {
    const double w = weight(i);
    r0 += cabs2(to_d2(gam[i])) * w;
    r1 += cabs2(to_d2(gam[i + ps])) * w;
  }
  r0 = group_sum_dpp(r0, 64);
  r1 = group_sum_dpp(r1, 64);
  if ((tid & 63) == 0) {
    red0[tid >> 6] = r0;
    red1[tid >> 6] = r1;
  }
  __syncthreads();
  double rho0 = 0.0, rho1 = 0.0;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) {
    rho0 += red0[w];
    rho1 += red1[w];
  }
  const double c = st.dldz[v];
  const double den = (rho0 + rho1) * (rho0 + rho1);
  const double d0 = c * 2.0 * rho1 / den, d1 = -c * 2.0 * rho0 / den;
  double2* gb = st.gbar + V.goff;
#pragma unroll 4
  for (int i = tid; i < ps; i += NT) {
    const double w = weight(i);
    const double2 a = to_d2(gam[i]), b = to_d2(gam[i + ps]);
    gb[i] = cscale(a, 2.0 * d0 * w);
    gb[i + ps] = cscale(b, 2.0 * d1 * w);
  }
  // dL/dW per leg index: for leg l and index k, the sum over the other legs' indices of
  // (d0 |G0|^2 + d1 |G1|^2) w.  The waves take the (l, k) bins in turn; lane j sums the bin's
  // elements j, j + 64, ... and a DPP wave sum adds the lanes, both in a fixed order, so the
  // gradient is bitwise reproducible.
  const int inner = deg ? ps / D : 0;
  const int lane = tid & 63;
  for (int bin = tid >> 6; bin < deg * D; bin += NT / 64) {
    const int l = bin / D, k = bin - (bin / D) * D;
    const int sl = l == 0 ? s0 : l == 1 ? s1 : 1;  // stride of leg l
    double sacc = 0.0;
    if (k < st.chi[V.leg[l]]) {  // the tensor is zero past a leg's active indices
#pragma unroll 4
      for (int j = lane; j < inner; j += 64) {
        const int hi = j / sl, lo = j - (j / sl) * sl;  // digits above and below leg l
        const int i = (hi * D + k) * sl + lo;
        sacc += (d0 * cabs2(to_d2(gam[i])) + d1 * cabs2(to_d2(gam[i + ps]))) * weight(i);
      }
    }
    sacc = group_sum_dpp(sacc, 64);
    if (lane == 0) acc[l][k] = sacc;
  }
  __syncthreads();
  for (int idx = tid; idx < deg * D; idx += NT) {
    const int l = idx / D, k = idx - (idx / D) * D;
    const double lam = st.lam[(int64_t)V.leg[l] * D + k];
    if (lam > 0.0 && acc[l][k] != 0.0) atomicAdd(&st.lbar[(int64_t)V.leg[l] * D + k], acc[l][k] * 2.0 / lam);
  }
}

// ------------------------------------------------------------------ RX adjoint

// Gamma' = RX Gamma on the physical index: Gamma-bar <- RX^H Gamma-bar,
// theta_h-bar += Re sum conj(Gamma'-bar) dRX Gamma with dRX = [[-s/2, -i c/2], [-i c/2, -s/2]].
template <typename CT>
__global__ __launch_bounds__(256) void k_adj_rx(DevState st, const void* __restrict__ pre, int chunk_first) {
  __shared__ double red[256];
  const int64_t ch = st.chunks[chunk_first + blockIdx.x];
  const int v = (int)(ch >> 32);
  const int cidx = (int)(ch & 0xffffffff);
  const VertexInfo& V = st.verts[v];
  const InstParam ip = st.inst[V.inst];
  int64_t ps = 1;
  for (int l = 0; l < V.deg; ++l) ps *= st.D;
  const CT* g0 = reinterpret_cast<const CT*>(pre) + V.goff;
  double2* gb = st.gbar + V.goff;
  const int64_t i0 = (int64_t)cidx * 1024;
  const double c = ip.rx_c, s = ip.rx_s;
  double part = 0.0;
  for (int64_t i = i0 + threadIdx.x; i < i0 + 1024 && i < ps; i += blockDim.x) {
    const double2 a = to_d2(g0[i]), b = to_d2(g0[i + ps]);
    const double2 ba = gb[i], bb = gb[i + ps];
    // dRX Gamma
    const double2 da = make_double2(-0.5 * s * a.x + 0.5 * c * b.y, -0.5 * s * a.y - 0.5 * c * b.x);
    const double2 db = make_double2(0.5 * c * a.y - 0.5 * s * b.x, -0.5 * c * a.x - 0.5 * s * b.y);
    part += cmulc(ba, da).x + cmulc(bb, db).x;
    // RX^H = [[c, i s], [i s, c]]
    gb[i] = make_double2(c * ba.x - s * bb.y, c * ba.y + s * bb.x);
    gb[i + ps] = make_double2(-s * ba.y + c * bb.x, s * ba.x + c * bb.y);
  }
  const double tot = block_sum<256>(part, red);
  // one workgroup per chunk: the chunk's own accumulator, summed per instance at the end
  if (threadIdx.x == 0) st.gpart[st.NE + chunk_first + blockIdx.x] += tot;
}

// ------------------------------------------------------------------ T-bar = Gamma^H Gamma'-bar

template <typename CT>
__global__ __launch_bounds__(256) void k_adj_tbar(DevState st, const int32_t* __restrict__ items, int first) {
  // T-bar[k][k'] = sum_m conj(Gamma[m][k]) Gamma'-bar[m][k'] on the FP64 matrix cores: with
  // v_mfma_f64_16x16x4f64 lane l holds A[l % 16][l / 16] and B[l / 16][l % 16] and receives
  // D[l / 16 + 4 r][l % 16], so the lane reads Gamma and Gamma'-bar at the same (row 4 s + l / 16,
  // column 16 t + l % 16) and the 16 lanes of a row read 16 consecutive columns.  Each wave sums a
  // quarter of the rows; the partial tiles are added in LDS in a fixed order.
  typedef double d4 __attribute__((ext_vector_type(4)));
  constexpr int NT16 = kMaxD / 16;  // column tiles of each operand
  constexpr int UNR = 4;            // row steps (of 4 rows) per load batch
  const int task = blockIdx.x;
  const int slot = task >> 2, side = (task >> 1) & 1, p = task & 1;
  const int e = items[first + slot];
  const SideInfo& S = st.edges[e].side[side];
  const int D = st.D;
  const SlotMeta meta = st.meta[slot];
  const int de = meta.de_old, chi = meta.chi_new;
  const int d1 = S.oth[0] >= 0 ? st.chi[S.oth[0]] : 1;
  const int d2 = S.oth[1] >= 0 ? st.chi[S.oth[1]] : 1;
  const int M = d1 * d2;
  const CT* gam = reinterpret_cast<const CT*>(st.gamma);
  const int64_t base = S.goff + p * S.pstride;
  const int tid = threadIdx.x, l = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6), li = l & 15, lk = l >> 4;
  const int ta_n = (de + 15) >> 4, tb_n = (chi + 15) >> 4;
  d4 cr[NT16][NT16], ci[NT16][NT16];
#pragma unroll
  for (int ta = 0; ta < NT16; ++ta)
#pragma unroll
    for (int tb = 0; tb < NT16; ++tb) {
      cr[ta][tb] = (d4){0.0, 0.0, 0.0, 0.0};
      ci[ta][tb] = (d4){0.0, 0.0, 0.0, 0.0};
    }
  const int ksteps = (M + 3) >> 2;
  // (rows and columns past the end are clamped, the loads do not wait for one another, and the
  // next batch loads during the products; the clamped rows are zeroed in Gamma when they are used,
  // clamped columns are not stored)
  CT na[UNR][NT16];
  double2 nb[UNR][NT16];
  auto fetch = [&](int ks0) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int m = min(4 * (ks0 + 4 * u) + lk, M - 1);
      const int o1 = m / d2, o2 = m - (m / d2) * d2;
      const int64_t ro = base + (int64_t)o1 * S.so[0] + (int64_t)o2 * S.so[1];
#pragma unroll
      for (int t = 0; t < NT16; ++t) {
        if (t < ta_n) na[u][t] = gam[ro + (int64_t)min(16 * t + li, de - 1) * S.sq];
        if (t < tb_n) nb[u][t] = st.gbar[ro + (int64_t)min(16 * t + li, chi - 1) * S.sq];
      }
    }
  };
  fetch(wv);
  for (int ks0 = wv; ks0 < ksteps; ks0 += 4 * UNR) {
    double2 ga[UNR][NT16], gb[UNR][NT16];
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const bool mv = 4 * (ks0 + 4 * u) + lk < M;
#pragma unroll
      for (int t = 0; t < NT16; ++t) {
        ga[u][t] = mv && t < ta_n ? to_d2(na[u][t]) : make_double2(0.0, 0.0);
        gb[u][t] = mv && t < tb_n ? nb[u][t] : make_double2(0.0, 0.0);
      }
    }
    if (ks0 + 4 * UNR < ksteps) fetch(ks0 + 4 * UNR);
#pragma unroll
    for (int u = 0; u < UNR; ++u)
#pragma unroll
      for (int ta = 0; ta < NT16; ++ta)
#pragma unroll
        for (int tb = 0; tb < NT16; ++tb) {
          if (ta < ta_n && tb < tb_n) {
            // conj(a) b = (a.x b.x + a.y b.y) + i (a.x b.y - a.y b.x)
            cr[ta][tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(ga[u][ta].x, gb[u][tb].x, cr[ta][tb], 0, 0, 0);
            cr[ta][tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(ga[u][ta].y, gb[u][tb].y, cr[ta][tb], 0, 0, 0);
            ci[ta][tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(ga[u][ta].x, gb[u][tb].y, ci[ta][tb], 0, 0, 0);
            ci[ta][tb] = __builtin_amdgcn_mfma_f64_16x16x4f64(-ga[u][ta].y, gb[u][tb].x, ci[ta][tb], 0, 0, 0);
          }
        }
  }
  // partial sums of the four waves, added in a fixed order: (0 + 2) + (1 + 3)
  __shared__ double2 part[2][NT16 * NT16 * 4][64];
  if (wv >= 2) {
#pragma unroll
    for (int ta = 0; ta < NT16; ++ta)
#pragma unroll
      for (int tb = 0; tb < NT16; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[wv - 2][(ta * NT16 + tb) * 4 + r][l] = make_double2(cr[ta][tb][r], ci[ta][tb][r]);
  }
  __syncthreads();
  if (wv < 2) {
#pragma unroll
    for (int ta = 0; ta < NT16; ++ta)
#pragma unroll
      for (int tb = 0; tb < NT16; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double2 q = part[wv][(ta * NT16 + tb) * 4 + r][l];
          cr[ta][tb][r] += q.x;
          ci[ta][tb][r] += q.y;
        }
  }
  __syncthreads();
  if (wv == 1) {
#pragma unroll
    for (int ta = 0; ta < NT16; ++ta)
#pragma unroll
      for (int tb = 0; tb < NT16; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[0][(ta * NT16 + tb) * 4 + r][l] = make_double2(cr[ta][tb][r], ci[ta][tb][r]);
  }
  __syncthreads();
  if (wv == 0) {
    double2* TB = st.wsb + (int64_t)slot * adj_scratch(D) + (int64_t)(side * 2 + p) * D * D;
#pragma unroll
    for (int ta = 0; ta < NT16; ++ta)
#pragma unroll
      for (int tb = 0; tb < NT16; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int k = 16 * ta + lk + 4 * r, kp = 16 * tb + li;
          if (k < de && kp < chi) {
            const double2 q = part[0][(ta * NT16 + tb) * 4 + r][l];
            TB[k * D + kp] = make_double2(cr[ta][tb][r] + q.x, ci[ta][tb][r] + q.y);
          }
        }
  }
}

// ------------------------------------------------------------------ small-matrix edge adjoint

// One small complex product C (+)= op(A) op(B), row-major, m x n with inner dimension k; op bit 0
// transposes, bit 1 conjugates (0 as is, 1 transpose, 2 conjugate, 3 conjugate transpose).
struct Gemm {
  int m, n, k;
  const double2* A;
  int lda, opA;
  const double2* B;
  int ldb, opB;
  double2* C;
  int ldc;
};

// This wave's number in its workgroup, the same on all its lanes.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

__device__ __forceinline__ int gemm_tiles(const Gemm& g) { return ((g.m + 15) >> 4) * ((g.n + 15) >> 4); }

typedef double adj_d4 __attribute__((ext_vector_type(4)));
typedef double adj_d2 __attribute__((ext_vector_type(2)));
// A descriptor's pointers come back from LDS, where the compiler loses that they are global ones:
// said here, or every access is a flat one, which also waits on LDS.
typedef __attribute__((address_space(1))) adj_d2 adj_mem;

// Adds the 16 x 16 tile (ti, tj) of g's product to (cr, ci), by one wave, on v_mfma_f64_16x16x4f64 (lane l
// holds A[l % 16][l / 16] and B[l / 16][l % 16] and receives D[l / 16 + 4 r][l % 16]), four real
// products per complex one; operands are read straight from memory, those of the next four k steps
// while the current ones are multiplied.  Indices past the end are clamped, so that no load waits for a
// branch or a select: rows and columns past m and n are not stored, and the products past k are
// zeroed in A when they are used.
__device__ __forceinline__ void gemm_acc(const Gemm& g, int ti, int tj, adj_d4& cr, adj_d4& ci) {
  const int l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
  const int K = __builtin_amdgcn_readfirstlane(g.k), ks = (K + 3) >> 2;
  const int i = min(16 * ti + li, g.m - 1), j = min(16 * tj + li, g.n - 1);
  const int sa = (g.opA & 1) ? g.lda : 1, sb = (g.opB & 1) ? 1 : g.ldb;  // strides of k
  const double ca = (g.opA & 2) ? -1.0 : 1.0, cb = (g.opB & 2) ? -1.0 : 1.0;
  const adj_mem* const A = (const adj_mem*)g.A + i * ((g.opA & 1) ? 1 : g.lda);
  const adj_mem* const B = (const adj_mem*)g.B + j * ((g.opB & 1) ? g.ldb : 1);
  adj_d4 er = {0.0, 0.0, 0.0, 0.0}, ei = {0.0, 0.0, 0.0, 0.0};
  adj_d2 na[4], nb[4];
  auto fetch = [&](int s0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int kk = min(4 * (s0 + u) + lk, K - 1);
      na[u] = A[kk * sa];
      nb[u] = B[kk * sb];
    }
  };
  if (K <= 0) return;
  fetch(0);
  for (int s0 = 0; s0 < ks; s0 += 4) {
    double2 a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double in = 4 * (s0 + u) + lk < K ? 1.0 : 0.0;
      a[u] = make_double2(in * na[u].x, in * ca * na[u].y);
      b[u] = make_double2(nb[u].x, cb * nb[u].y);
    }
    if (s0 + 4 < ks) fetch(s0 + 4);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (s0 + u < ks) {
        cr = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].x, b[u].x, cr, 0, 0, 0);
        ci = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].x, b[u].y, ci, 0, 0, 0);
        er = __builtin_amdgcn_mfma_f64_16x16x4f64(-a[u].y, b[u].y, er, 0, 0, 0);
        ei = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].y, b[u].x, ei, 0, 0, 0);
      }
    }
  }
  cr += er;
  ci += ei;
}

__device__ __forceinline__ void gemm_store(const Gemm& g, int ti, int tj, const adj_d4& cr, const adj_d4& ci,
                                           bool accumulate) {
  const int l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
  adj_mem* const C = (adj_mem*)g.C;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int ii = 16 * ti + lk + 4 * r, jj = 16 * tj + li;
    if (ii < g.m && jj < g.n) {
      const adj_d2 v = {cr[r], ci[r]};
      C[ii * g.ldc + jj] = accumulate ? C[ii * g.ldc + jj] + v : v;
    }
  }
}

__device__ __forceinline__ void gemm_tile(const Gemm& g, int tile, bool accumulate) {
  const int tn = (g.n + 15) >> 4;
  const int ti = tile / tn, tj = tile - (tile / tn) * tn;
  adj_d4 cr = {0.0, 0.0, 0.0, 0.0}, ci = {0.0, 0.0, 0.0, 0.0};
  gemm_acc(g, ti, tj, cr, ci);
  gemm_store(g, ti, tj, cr, ci, accumulate);
}

// NG mutually independent products: their output tiles are spread over the waves of the block
// together, then one barrier.  The descriptors go through LDS (`gd`, at least NG entries, not
// in use by another batch), so each tile reads its product's descriptor with a uniform index.
template <int NG>
__device__ void bgemm_batch(const Gemm (&gs)[NG], Gemm* gd, bool accumulate) {
  if (threadIdx.x == 0) {
#pragma unroll
    for (int i = 0; i < NG; ++i) gd[i] = gs[i];
  }
  int tot = 0;
#pragma unroll
  for (int i = 0; i < NG; ++i) tot += gemm_tiles(gs[i]);
  __syncthreads();
  for (int tile = wave_id(); tile < tot; tile += (int)(blockDim.x >> 6)) {
    int i = 0, t = tile;
    while (t >= gemm_tiles(gd[i])) {
      t -= gemm_tiles(gd[i]);
      ++i;
    }
    const Gemm g = gd[i];
    gemm_tile(g, t, accumulate);
  }
  __syncthreads();
}

__device__ void bgemm(const Gemm& g, bool accumulate) {
  for (int tile = wave_id(); tile < gemm_tiles(g); tile += (int)(blockDim.x >> 6))
    gemm_tile(g, tile, accumulate);
  __syncthreads();
}

// C = g + h, two products into one output (g's).
__device__ void bgemm_sum(const Gemm& g, const Gemm& h) {
  const int tn = (g.n + 15) >> 4;
  for (int tile = wave_id(); tile < gemm_tiles(g); tile += (int)(blockDim.x >> 6)) {
    const int ti = tile / tn, tj = tile - (tile / tn) * tn;
    adj_d4 cr = {0.0, 0.0, 0.0, 0.0}, ci = {0.0, 0.0, 0.0, 0.0};
    gemm_acc(g, ti, tj, cr, ci);
    gemm_acc(h, ti, tj, cr, ci);
    gemm_store(g, ti, tj, cr, ci, false);
  }
  __syncthreads();
}

// x of the lane `lane` (the same on every lane).
__device__ __forceinline__ double lane_value(double x, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                          __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// REC: the forward recovered one singular-vector set as Theta' v / sigma (complex64 path), which
// is accurate only to ~2^-52 s_0 / sigma.  Triplets at that noise level (sigma <= kRecTau s_0) are
// then left out of the F terms and their directions go with the orthogonal complement of the
// retained ones, weighted s_k / (s_k^2 + eps_F s_0^2): the value the F term itself takes for a
// partner of vanishing sigma.  A noise-level triplet thus contributes the same whether it is
// retained or not, and the result does not depend on how the forward resolved them.  Without
// REC (both sets accumulated, complex128) every triplet above 1e-13 s_0 is retained and the
// complement takes 1 / s_k.
//
// N bounds D (16 or 32).  One workgroup per edge and few edges a launch: bound by the latency of its
// chain of small products, so the operands of the next k steps are in flight during the current ones,
// eight waves share the tiles of a batch, and the eliminations run in registers.
// Mean over the classes of the 127-qubit graph (one instance): 86 -> 47 us at D = 16, 163 -> 85 us at
// D = 32; a four-wave form that waited for every pair of loads and eliminated in LDS is the first figure.
constexpr int kSmallThreads = 512;

template <bool REC, int N>
__global__ __launch_bounds__(kSmallThreads) void k_adj_small(DevState st, const int32_t* __restrict__ items, int first,
                                                             double2* __restrict__ ybuf) {
  __shared__ double red[kSmallThreads];
  __shared__ double Sv[2 * N], Sb[2 * N], Lb[N], lam[N], Lo[N];
  __shared__ int sh_rp;
  __shared__ double Pt[N][N + 1];      // elementwise products, reduced by rows / columns
  __shared__ double2 Yt[4][N][N + 1];  // Y of the four QR backwards
  __shared__ Gemm gdesc[8];                            // descriptors of a batch of small products
  const int slot = blockIdx.x;
  const int e = items[first + slot];
  const EdgeInfo& E = st.edges[e];
  const InstParam ip = st.inst[E.inst];
  const int D = st.D, NM = 2 * D;
  const int tid = threadIdx.x;
  const SlotMeta meta = st.meta[slot];
  const int de = meta.de_old, chi = meta.chi_new;
  int r[2], Ms[2];
  for (int sd = 0; sd < 2; ++sd) {
    const SideInfo& S = E.side[sd];
    const int d1 = S.oth[0] >= 0 ? st.chi[S.oth[0]] : 1;
    const int d2 = S.oth[1] >= 0 ? st.chi[S.oth[1]] : 1;
    Ms[sd] = d1 * d2;
    r[sd] = min(Ms[sd], de);
  }
  const int ri = r[0], rj = r[1], m0 = 2 * ri, n0 = 2 * rj;
  const int rr = min(m0, n0);
  const int64_t q = (int64_t)D * D;
  double2* base = st.wsb + (int64_t)slot * adj_scratch(D);
  double2* TB = base;
  double2* Ub = base + 4 * q;
  double2* Vb = base + 8 * q;
  double2* J = base + 12 * q;
  double2* K = base + 16 * q;
  double2* In = base + 20 * q;
  double2* M1 = base + 24 * q;
  double2* Vp = base + 28 * q;
  double2* Thb = base + 32 * q;
  double2* X = base + 36 * q;
  double2* Yc = base + 38 * q;
  double2* Xb = base + 40 * q;
  double2* Ycb = base + 42 * q;
  double2* Rb = base + 44 * q;
  double2* H = base + 12 * q;  // [4][D][D] reuses J after the SVD backward
  const double2* U = st.bU + (int64_t)slot * NM * NM;
  const double2* V = st.bV + (int64_t)slot * NM * NM;
  const double2* Rg = st.rbuf + rbuf_off(st, slot, 0, 0);  // i0, i1, j0, j1 blocks of D*D
  const double2* T64 = st.t64 + rbuf_off(st, slot, 0, 0);
  double2* Yout = ybuf + rbuf_off(st, slot, 0, 0);
  const double* lam_g = st.lam + (int64_t)e * D;
  double* lbar_e = st.lbar + (int64_t)e * D;
  const double2 g[2][2] = {{gate_phase(ip, 0, 0), gate_phase(ip, 0, 1)}, {gate_phase(ip, 1, 0), gate_phase(ip, 1, 1)}};
  const double2 dg[2][2] = {{gate_dphase(ip, 0, 0), gate_dphase(ip, 0, 1)},
                            {gate_dphase(ip, 1, 0), gate_dphase(ip, 1, 1)}};

  for (int k = tid; k < rr; k += blockDim.x) Sv[k] = st.bS[(int64_t)slot * NM + k];
  for (int k = tid; k < N; k += blockDim.x) {
    lam[k] = k < de ? lam_g[k] : 0.0;
    Lo[k] = k < chi ? lbar_e[k] : 0.0;
  }
  if (tid < 64) {  // rr <= 2 N <= 64
    const double tau = REC ? kRecTau : 1e-13;
    const double s = tid < rr ? st.bS[(int64_t)slot * NM + tid] : 0.0;
    const int rp = __popcll(__ballot(tid < rr && s > tau * lane_value(s, 0)));
    if (tid == 0) sh_rp = rp > chi ? rp : chi;
  }
  __syncthreads();
  const int rp = sh_rp;
  double thj = 0.0;

  // lambda' = S_chi / ||S_chi||  ->  S-bar;  T terms -> S-bar, lambda-bar
  double nrm2 = 0.0, ls = 0.0;
  for (int k = 0; k < chi; ++k) {
    nrm2 += Sv[k] * Sv[k];
    ls += Lo[k] * Sv[k];
  }
  const double nrm = sqrt(nrm2);
  // P[k][k'] = sum_w Re conj(TB_w[k][k']) T64_w[k][k'] in parallel, then its column sums give
  // the T terms of S-bar and its row sums those of lambda-bar
  for (int idx = tid; idx < de * chi; idx += blockDim.x) {
    const int k = idx / chi, kp = idx - (idx / chi) * chi;
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) t += cmulc(TB[w * q + k * D + kp], T64[w * q + k * D + kp]).x;
    Pt[k][kp] = t;
  }
  __syncthreads();
  for (int kp = tid; kp < rr; kp += blockDim.x) {
    double sb = 0.0;
    if (kp < chi) {
      sb = Lo[kp] / nrm - Sv[kp] * ls / (nrm2 * nrm);
      double t = 0.0;
      for (int k = 0; k < de; ++k) t += Pt[k][kp];
      sb -= t / Sv[kp];
    }
    Sb[kp] = sb;
  }
  for (int k = tid; k < de; k += blockDim.x) {
    double t = 0.0;
    for (int kp = 0; kp < chi; ++kp) t += Pt[k][kp];
    Lb[k] = t / lam[k];
  }
  // X_t = R_j^(t)T V_t[:, :chi],  Yc_s = R_i^(s)T conj(U_s[:, :chi])
  {
    const Gemm gs[4] = {{de, chi, rj, Rg + 2 * q, D, 1, V, NM, 0, X, D},
                        {de, chi, rj, Rg + 3 * q, D, 1, V + rj * NM, NM, 0, X + q, D},
                        {de, chi, ri, Rg, D, 1, U, NM, 2, Yc, D},
                        {de, chi, ri, Rg + q, D, 1, U + ri * NM, NM, 2, Yc + q, D}};
    bgemm_batch(gs, gdesc, false);
  }
  // theta_J and the adjoints of X, Yc
  for (int idx = tid; idx < de * chi; idx += blockDim.x) {
    const int k = idx / chi, kp = idx - (idx / chi) * chi;
    const double f = lam[k] / Sv[kp];
    for (int t = 0; t < 2; ++t) {
      double2 xb = make_double2(0.0, 0.0), ycb = make_double2(0.0, 0.0);
      for (int s = 0; s < 2; ++s) {
        xb = cadd(xb, cmulc(g[s][t], TB[s * q + k * D + kp]));
        ycb = cadd(ycb, cmulc(g[t][s], TB[(2 + s) * q + k * D + kp]));
      }
      Xb[t * q + k * D + kp] = cscale(xb, f);    // sum_s conj(g(s,t)) lambda_k TB_i^(s) / s_k'
      Ycb[t * q + k * D + kp] = cscale(ycb, f);  // (index t here is s): sum_t conj(g(s,t)) lambda TB_j^(t) / s
    }
    for (int s = 0; s < 2; ++s) {
      double2 a = make_double2(0.0, 0.0), b = make_double2(0.0, 0.0);
      for (int t = 0; t < 2; ++t) {
        a = cadd(a, cmul(dg[s][t], X[t * q + k * D + kp]));
        b = cadd(b, cmul(dg[t][s], Yc[t * q + k * D + kp]));
      }
      thj += f * (cmulc(TB[s * q + k * D + kp], a).x + cmulc(TB[(2 + s) * q + k * D + kp], b).x);
    }
  }
  __syncthreads();
  // R-bar_j^(t) = Xb_t^T... : R-bar_j^(t)[b,k] = sum_k' Xb_t[k,k'] conj(V_t[b,k']);  V-bar_t = conj(R_j^(t)) Xb_t
  {
    const Gemm gs[8] = {{rj, de, chi, V, NM, 2, Xb, D, 1, Rb + 2 * q, D},
                        {rj, chi, de, Rg + 2 * q, D, 2, Xb, D, 0, Vb, NM},
                        {rj, de, chi, V + rj * NM, NM, 2, Xb + q, D, 1, Rb + 3 * q, D},
                        {rj, chi, de, Rg + 3 * q, D, 2, Xb + q, D, 0, Vb + rj * NM, NM},
                        {ri, de, chi, U, NM, 0, Ycb, D, 1, Rb, D},
                        {ri, chi, de, Rg, D, 0, Ycb, D, 2, Ub, NM},
                        {ri, de, chi, U + ri * NM, NM, 0, Ycb + q, D, 1, Rb + q, D},
                        {ri, chi, de, Rg + q, D, 0, Ycb + q, D, 2, Ub + ri * NM, NM}};
    bgemm_batch(gs, gdesc, false);
  }
  // zero the columns chi..rp-1 of U-bar, V-bar
  for (int idx = tid; idx < m0 * (rp - chi); idx += blockDim.x) {
    const int a = idx / (rp - chi), c = chi + idx - (idx / (rp - chi)) * (rp - chi);
    Ub[a * NM + c] = make_double2(0.0, 0.0);
  }
  for (int idx = tid; idx < n0 * (rp - chi); idx += blockDim.x) {
    const int a = idx / (rp - chi), c = chi + idx - (idx / (rp - chi)) * (rp - chi);
    Vb[a * NM + c] = make_double2(0.0, 0.0);
  }
  __syncthreads();

  // ---- complex SVD backward over the rp triplets with s > 1e-13 s_0
  {
    const Gemm gs[2] = {{rp, rp, m0, U, NM, 3, Ub, NM, 0, J, NM}, {rp, rp, n0, V, NM, 3, Vb, NM, 0, K, NM}};
    bgemm_batch(gs, gdesc, false);
  }
  const double s0 = Sv[0];
  for (int idx = tid; idx < rp * rp; idx += blockDim.x) {
    const int k = idx / rp, l = idx - (idx / rp) * rp;
    double2 v;
    if (k == l) {
      const double im = (k < chi) ? 0.5 * (J[k * NM + k].y - K[k * NM + k].y) / Sv[k] : 0.0;
      v = make_double2(Sb[k], im);
    } else {
      const double sk = Sv[k] / s0, sl = Sv[l] / s0;
      const double d = sl - sk, ss = sk + sl;
      const double f = ss > 0.0 ? d / (d * d + kEpsF) / ss / (s0 * s0) : 0.0;
      const double2 aj = csub(J[k * NM + l], cconj(J[l * NM + k]));
      const double2 ak = csub(K[k * NM + l], cconj(K[l * NM + k]));
      v = cadd(cscale(aj, f * Sv[l]), cscale(ak, f * Sv[k]));
    }
    In[k * NM + l] = v;
  }
  __syncthreads();
  // U-bar' = (U-bar - U J) S^-1 and V-bar' = (V-bar - V K) S^-1 on the kept columns
  {
    const Gemm gs[2] = {{m0, rp, rp, U, NM, 0, J, NM, 0, M1, NM}, {n0, rp, rp, V, NM, 0, K, NM, 0, Vp, NM}};
    bgemm_batch(gs, gdesc, false);
  }
  // weight of the orthogonal complement of the retained triplets (see REC above)
  auto cw = [&](int l) { return REC ? Sv[l] / (Sv[l] * Sv[l] + kEpsF * s0 * s0) : 1.0 / Sv[l]; };
  for (int idx = tid; idx < m0 * rp; idx += blockDim.x) {
    const int a = idx / rp, l = idx - (idx / rp) * rp;
    M1[a * NM + l] = l < chi ? cscale(csub(Ub[a * NM + l], M1[a * NM + l]), cw(l)) : make_double2(0.0, 0.0);
  }
  for (int idx = tid; idx < n0 * rp; idx += blockDim.x) {
    const int a = idx / rp, l = idx - (idx / rp) * rp;
    Vp[a * NM + l] = l < chi ? cscale(csub(Vb[a * NM + l], Vp[a * NM + l]), cw(l)) : make_double2(0.0, 0.0);
  }
  __syncthreads();
  // M1 += U In ;  Theta'-bar = M1 V^H + U Vp^H
  bgemm({m0, rp, rp, U, NM, 0, In, NM, 0, M1, NM}, true);
  bgemm_sum({m0, n0, rp, M1, NM, 0, V, NM, 3, Thb, NM}, {m0, n0, rp, U, NM, 0, Vp, NM, 3, Thb, NM});

  // ---- Theta' backward: H_st = Thb_st conj(R_j^(t))  [ri x de]
  {
    const Gemm gs[4] = {{ri, de, rj, Thb, NM, 0, Rg + 2 * q, D, 2, H, D},
                        {ri, de, rj, Thb + rj, NM, 0, Rg + 3 * q, D, 2, H + q, D},
                        {ri, de, rj, Thb + ri * NM, NM, 0, Rg + 2 * q, D, 2, H + 2 * q, D},
                        {ri, de, rj, Thb + ri * NM + rj, NM, 0, Rg + 3 * q, D, 2, H + 3 * q, D}};
    bgemm_batch(gs, gdesc, false);
  }
  for (int idx = tid; idx < ri * de; idx += blockDim.x) {
    const int a = idx / de, k = idx - (idx / de) * de;
    double lt = 0.0;  // this (a, k)'s share of lambda-bar_k
    for (int s = 0; s < 2; ++s) {
      double2 acc = make_double2(0.0, 0.0);
      const double2 rik = Rg[s * q + a * D + k];
      for (int t = 0; t < 2; ++t) {
        const double2 h = H[(s * 2 + t) * q + a * D + k];
        acc = cadd(acc, cmulc(g[s][t], h));
        thj += lam[k] * cmulc(h, cmul(dg[s][t], rik)).x;
        lt += cmulc(h, cmul(g[s][t], rik)).x;
      }
      Rb[s * q + a * D + k] = cadd(Rb[s * q + a * D + k], cscale(acc, lam[k]));
    }
    Pt[a][k] = lt;
  }
  __syncthreads();
  for (int k = tid; k < de; k += blockDim.x) {
    double t = 0.0;
    for (int a = 0; a < ri; ++a) t += Pt[a][k];
    Lb[k] += t;
  }
  __syncthreads();
  // R-bar_j^(t)[b,k] += lambda_k sum_s conj(g(s,t)) P_st[b,k], P_st = Thb_st^T conj(R_i^(s)) [rj x de]
  // (P_st in the H region, which the loops above have finished with)
  {
    const Gemm gs[4] = {{rj, de, ri, Thb, NM, 1, Rg, D, 2, H, D},
                        {rj, de, ri, Thb + rj, NM, 1, Rg, D, 2, H + q, D},
                        {rj, de, ri, Thb + ri * NM, NM, 1, Rg + q, D, 2, H + 2 * q, D},
                        {rj, de, ri, Thb + ri * NM + rj, NM, 1, Rg + q, D, 2, H + 3 * q, D}};
    bgemm_batch(gs, gdesc, false);
  }
  for (int idx = tid; idx < rj * de; idx += blockDim.x) {
    const int b = idx / de, k = idx - (idx / de) * de;
    for (int t = 0; t < 2; ++t) {
      double2 acc = make_double2(0.0, 0.0);
      for (int s = 0; s < 2; ++s) acc = cadd(acc, cmulc(g[s][t], H[(s * 2 + t) * q + b * D + k]));
      Rb[(2 + t) * q + b * D + k] = cadd(Rb[(2 + t) * q + b * D + k], cscale(acc, lam[k]));
    }
  }
  __syncthreads();

  // ---- QR backward of the four (end, slice) blocks, solved together.  A block that was not
  // reduced (M <= D_e, R = A) has A-bar = R-bar.  For the others G = R^H R and Z = R^H R-bar
  // (one batch of products; G in the H region, finished with above), then
  // Y = (G + delta I)^-1 Z by Gauss-Jordan elimination of [G + delta I | Z] (Hermitian positive
  // definite: no pivoting), one wave per block and one lane per column with the column in
  // registers, so the four run side by side with no workgroup barrier.
  bool redw[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) redw[w] = Ms[w >> 1] > de;
  for (int w = 0; w < 4; ++w) {
    if (redw[w]) continue;
    const int rows = (w >> 1) ? rj : ri;
    for (int idx = tid; idx < rows * de; idx += blockDim.x) {
      const int a = idx / de, k = idx - (idx / de) * de;
      Yout[w * q + a * D + k] = Rb[w * q + a * D + k];
    }
    if (tid == 0) st.ymode[slot * 4 + w] = 1;
  }
  {
    const int n0r = redw[0] ? de : 0, n1r = redw[1] ? de : 0, n2r = redw[2] ? de : 0, n3r = redw[3] ? de : 0;
    const Gemm gs[8] = {{n0r, de, ri, Rg, D, 3, Rg, D, 0, H, D},
                        {n0r, de, ri, Rg, D, 3, Rb, D, 0, Yout, D},
                        {n1r, de, ri, Rg + q, D, 3, Rg + q, D, 0, H + q, D},
                        {n1r, de, ri, Rg + q, D, 3, Rb + q, D, 0, Yout + q, D},
                        {n2r, de, rj, Rg + 2 * q, D, 3, Rg + 2 * q, D, 0, H + 2 * q, D},
                        {n2r, de, rj, Rg + 2 * q, D, 3, Rb + 2 * q, D, 0, Yout + 2 * q, D},
                        {n3r, de, rj, Rg + 3 * q, D, 3, Rg + 3 * q, D, 0, H + 3 * q, D},
                        {n3r, de, rj, Rg + 3 * q, D, 3, Rb + 3 * q, D, 0, Yout + 3 * q, D}};
    bgemm_batch(gs, gdesc, false);
  }
  {
    // wave w solves system w; lane c owns column c of [G | Z] (G: c < de, Z: N <= c < N + de).  Before
    // step p, x[i] is row (p + i) % N: the pivot row is always x[0] and each step moves the rows up
    // by one, so that one copy of the step serves all (rows from de on stay zero).
    const int wq = tid >> 6, lc = tid & 63;
    if (wq < 4 && redw[wq]) {
      const bool gcol = lc < de, zcol = lc >= N && lc < N + de;
      const double2* src = gcol ? H + wq * q + lc : Yout + wq * q + (zcol ? lc - N : 0);
      double2 x[N];
      double dmax = 0.0;
#pragma unroll
      for (int a = 0; a < N; ++a) {
        x[a] = a < de ? src[a * D] : make_double2(0.0, 0.0);
        if (!gcol && !zcol) x[a] = make_double2(0.0, 0.0);
        if (gcol && a == lc) dmax = x[a].x;
      }
      dmax = wave_max(dmax);
      const double delta = 1e-13 * (dmax > 0.0 ? dmax : 1.0);
#pragma unroll
      for (int a = 0; a < N; ++a)
        if (gcol && a == lc) x[a].x += delta;
      for (int p = 0; p < de; ++p) {
        // scale the pivot row by 1 / G[p][p] (real: Hermitian), then eliminate column p from the others
        const double ip = 1.0 / lane_value(x[0].x, p);
        const double2 rpc = cscale(x[0], ip);
#pragma unroll
        for (int i = 1; i < N; ++i) {
          const double2 f = make_double2(lane_value(x[i].x, p), lane_value(x[i].y, p));
          x[i - 1] = csub(x[i], cmul(f, rpc));
        }
        x[N - 1] = rpc;
      }
      // Hermitian part of Y; row a ended at x[N - de + a]
#pragma unroll
      for (int i = 0; i < N; ++i)
        if (zcol && i >= N - de) Yt[wq][i - (N - de)][lc - N] = x[i];
      wave_lds_sync();
      if (zcol) {
        const int b = lc - N;
        for (int a = 0; a < de; ++a) {
          double2 h = cscale(cadd(Yt[wq][a][b], cconj(Yt[wq][b][a])), 0.5);
          if (a == b) h.y = 0.0;
          Yout[wq * q + a * D + b] = h;
        }
      }
      if (lc == 0) st.ymode[slot * 4 + wq] = 0;
    }
  }
  __syncthreads();

  // ---- pre-gate lambda_e adjoint and dL/dtheta_J
  for (int k = tid; k < D; k += blockDim.x) lbar_e[k] = k < de ? Lb[k] : 0.0;
  const double tot = block_sum<kSmallThreads>(thj, red);
  // one item per edge in a launch: the edge's own accumulator, summed per instance at the end
  if (tid == 0) st.gpart[e] += tot;
}

// ------------------------------------------------------------------ Gamma-bar rows

// Gamma-bar = Gamma'-bar T^H + w A-bar and w-bar = sum_k Re conj(A-bar) Gamma per row, with
// A-bar = w (Gamma Y) or, where the slice was not reduced, the stored R-bar.  Each wave takes 16 rows and
// every column: both products on v_mfma_f64_16x16x4f64 (lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16] and receives D[l / 16 + 4 r][l % 16]), operands from memory to registers (T and Y
// from the caches), no LDS and no barrier.  Clamped indices as in gemm_acc.  Bound by latency at
// D = 16 and by the FP64 matrix cores above.  N bounds D.  One class
// of the 127-qubit graph (mean): 13.9 -> 9.4 us at D = 16, 59.8 -> 28.2 us at D = 32 against vector dot
// products on rows staged in LDS.
template <typename CT, int N>
__global__ __launch_bounds__(256, N == 32 ? 2 : 4) void k_adj_rows(DevState st, const int32_t* __restrict__ items, int first,
                                                  int blocks_per_slice, const double2* __restrict__ ybuf) {
  constexpr int NT = N / 16;
  int slot, sp, rb;
  row_task(st, blockIdx.x, blocks_per_slice, slot, sp, rb);
  const int side = sp >> 1, p = sp & 1;
  const int e = items[first + slot];
  const SideInfo& S = st.edges[e].side[side];
  const int D = st.D;
  const int d1 = S.oth[0] >= 0 ? st.chi[S.oth[0]] : 1;
  const int d2 = S.oth[1] >= 0 ? st.chi[S.oth[1]] : 1;
  const int M = d1 * d2;
  static_assert(kRowBlock == 4 * 16, "16 rows a wave");
  const int row0 = rb * kRowBlock + 16 * __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (row0 >= M) return;
  const SlotMeta meta = st.meta[slot];
  const int de = meta.de_old, chi = meta.chi_new;
  const int ncol = max(de, chi);
  const bool reduced = st.ymode[slot * 4 + sp] == 0;
  const double* l1 = S.oth[0] >= 0 ? st.lam + (int64_t)S.oth[0] * D : nullptr;
  const double* l2 = S.oth[1] >= 0 ? st.lam + (int64_t)S.oth[1] * D : nullptr;
  const double2* T = st.t64 + rbuf_off(st, slot, side, p);
  const double2* Y = ybuf + rbuf_off(st, slot, side, p);
  const int64_t base = S.goff + p * S.pstride, so0 = S.so[0], so1 = S.so[1], sq = S.sq;
  const CT* gam = reinterpret_cast<const CT*>(st.gamma);
  double2* const gbar = st.gbar;
  const int l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
  auto row_off = [&](int m) -> int64_t {
    const int o1 = m / d2, o2 = m - (m / d2) * d2;
    return base + o1 * so0 + o2 * so1;
  };
  const int64_t ra = row_off(min(row0 + li, M - 1));
  // Gamma at the output positions and the rows' weights, in flight during the products
  CT gout[4][NT];
  double w[4];
  int64_t ro[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = min(row0 + lk + 4 * r, M - 1);
    const int o1 = m / d2, o2 = m - (m / d2) * d2;
    ro[r] = base + o1 * so0 + o2 * so1;
    w[r] = (l1 ? l1[o1] : 1.0) * (l2 ? l2[o2] : 1.0);
#pragma unroll
    for (int t = 0; t < NT; ++t)
      if (16 * t < de) gout[r][t] = gam[ro[r] + min(16 * t + li, de - 1) * sq];
  }
  adj_d4 br[NT], bi[NT], yr[NT], yi[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    br[t] = (adj_d4){0.0, 0.0, 0.0, 0.0};
    bi[t] = br[t];
    yr[t] = br[t];
    yi[t] = br[t];
  }
#pragma unroll
  for (int k0 = 0; k0 < N; k0 += 16) {
    if (k0 < chi) {  // Gamma'-bar T^H over k' = k0 .. k0 + 15
      double2 x[4], y[4][NT];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int kp = min(k0 + 4 * u + lk, chi - 1);
        x[u] = gbar[ra + kp * sq];
#pragma unroll
        for (int t = 0; t < NT; ++t)
          if (16 * t < de) y[u][t] = T[min(16 * t + li, de - 1) * D + kp];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double2 a = k0 + 4 * u + lk < chi ? x[u] : make_double2(0.0, 0.0);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          if (16 * t < de && k0 + 4 * u < chi) {
            const double2 b = y[u][t];  // conjugated
            br[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, br[t], 0, 0, 0);
            bi[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, bi[t], 0, 0, 0);
            br[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.y, br[t], 0, 0, 0);
            bi[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.x, b.y, bi[t], 0, 0, 0);
          }
      }
    }
    if (reduced && k0 < de) {  // Gamma Y
      CT x[4];
      double2 y[4][NT];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = min(k0 + 4 * u + lk, de - 1);
        x[u] = gam[ra + k * sq];
#pragma unroll
        for (int t = 0; t < NT; ++t)
          if (16 * t < de) y[u][t] = Y[k * D + min(16 * t + li, de - 1)];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const double2 a = k0 + 4 * u + lk < de ? to_d2(x[u]) : make_double2(0.0, 0.0);
#pragma unroll
        for (int t = 0; t < NT; ++t)
          if (16 * t < de && k0 + 4 * u < de) {
            const double2 b = y[u][t];
            yr[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.x, yr[t], 0, 0, 0);
            yi[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b.y, yi[t], 0, 0, 0);
            yr[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, b.y, yr[t], 0, 0, 0);
            yi[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b.x, yi[t], 0, 0, 0);
          }
      }
    }
  }
  // the wave's rows have been read: Gamma-bar goes out in place, w-bar per row (w = l1[o1] l2[o2]) to
  // k_adj_lbar, which folds it into the other legs' lambda-bar
  double ws[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = row0 + lk + 4 * r;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int k = 16 * t + li;
      if (m < M && k < ncol) {
        double2 out = make_double2(0.0, 0.0);
        if (k < de) {
          const double2 abar = reduced ? make_double2(w[r] * yr[t][r], w[r] * yi[t][r]) : Y[m * D + k];
          out = make_double2(fma(w[r], abar.x, br[t][r]), fma(w[r], abar.y, bi[t][r]));
          ws[r] += cmulc(abar, to_d2(gout[r][t])).x;
        }
        gbar[ro[r] + k * sq] = out;
      }
    }
  }
  double* wrow = st.wbar + ((int64_t)slot * 4 + sp) * D * D;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double v = group_sum_dpp(ws[r], 16);
    const int m = row0 + lk + 4 * r;
    if (li == 0 && m < M) wrow[m] = v;
  }
}

// lambda-bar of the other legs of one end (slot, side) from the per-row w-bar of both slices:
//   lambda-bar[f1][o1] += sum_p sum_o2 wbar[p][o1 d2 + o2] l2[o2],
//   lambda-bar[f2][o2] += sum_p sum_o1 wbar[p][o1 d2 + o2] l1[o1],
// summed in a fixed order.  An edge f gets such terms from the ends at its two vertices; pass 0
// adds the term of its lower vertex, pass 1 that of its higher one, so the additions into
// lambda-bar[f] happen in one order on every run.  Bound by its chain of dependent loads: 6.3 -> 4.6 us a
// pass with eight lanes an entry instead of one.
__global__ __launch_bounds__(256) void k_adj_lbar(DevState st, const int32_t* __restrict__ items, int first,
                                                  int pass) {
  const int slot = blockIdx.x >> 1, side = blockIdx.x & 1;
  const int e = items[first + slot];
  const SideInfo& S = st.edges[e].side[side];
  const int D = st.D;
  const int d1 = S.oth[0] >= 0 ? st.chi[S.oth[0]] : 1;
  const int d2 = S.oth[1] >= 0 ? st.chi[S.oth[1]] : 1;
  const double* l1 = S.oth[0] >= 0 ? st.lam + (int64_t)S.oth[0] * D : nullptr;
  const double* l2 = S.oth[1] >= 0 ? st.lam + (int64_t)S.oth[1] * D : nullptr;
  const double* w0 = st.wbar + ((int64_t)slot * 4 + side * 2 + 0) * D * D;
  const double* w1 = st.wbar + ((int64_t)slot * 4 + side * 2 + 1) * D * D;
  const int tid = threadIdx.x;
  for (int leg = 0; leg < 2; ++leg) {
    const int f = S.oth[leg];
    if (f < 0) continue;
    const bool lower = st.edges[f].side[0].goff == S.goff;
    if (lower != (pass == 0)) continue;
    // eight lanes an entry o (256 / 8 = kMaxD entries), their shares added in a fixed order
    static_assert(8 * kMaxD == 256, "eight lanes an entry");
    const int n = leg == 0 ? d1 : d2, m = leg == 0 ? d2 : d1;
    const int so = leg == 0 ? d2 : 1, sj = leg == 0 ? 1 : d2;
    const double* lo = leg == 0 ? l2 : l1;
    const int o = tid >> 3;
    double acc = 0.0;
#pragma unroll
    for (int u = 0; u < kMaxD / 8; ++u) {
      const int j = (tid & 7) + 8 * u;
      if (o < n && j < m) acc += (w0[o * so + j * sj] + w1[o * so + j * sj]) * (lo ? lo[j] : 1.0);
    }
    acc = group_sum_dpp(acc, 8);
    if ((tid & 7) == 0 && o < n && acc != 0.0) st.lbar[(int64_t)f * D + o] += acc;
  }
}

// dL/dtheta of every instance from the per-edge (theta_J) and per-chunk (theta_h) accumulators,
// each summed in a fixed order (thread stride, then a fixed tree).
__global__ __launch_bounds__(256) void k_adj_theta(DevState st, int n_chunks) {
  __shared__ double red[256];
  const int k = blockIdx.x;
  double tj = 0.0, th = 0.0;
  for (int e = threadIdx.x; e < st.NE; e += 256)
    if (st.edges[e].inst == k) tj += st.gpart[e];
  for (int c = threadIdx.x; c < n_chunks; c += 256)
    if (st.verts[(int)(st.chunks[c] >> 32)].inst == k) th += st.gpart[st.NE + c];
  const double sj = block_sum<256>(tj, red);
  const double sh = block_sum<256>(th, red);
  if (threadIdx.x == 0) {
    st.thbar[2 * k + 0] = sh;
    st.thbar[2 * k + 1] = sj;
  }
}

// ------------------------------------------------------------------ launchers

template <typename CT>
static hipError_t adj_launch(int which, const DevState& st, const int32_t* items, int first, int count,
                             int blocks_per_slice, const void* aux, hipStream_t stream) {
  switch (which) {
    case 1:
      if (count <= 0) return hipSuccess;
      hipLaunchKernelGGL(k_adj_tbar<CT>, dim3(count * 4), dim3(256), 0, stream, st, items, first);
      break;
    case 2:
      if (count <= 0) return hipSuccess;
      {
        constexpr bool kRec = std::is_same<CT, float2>::value;
        const auto kern = st.D <= 16 ? k_adj_small<kRec, 16> : k_adj_small<kRec, 32>;
        hipLaunchKernelGGL(kern, dim3(count), dim3(kSmallThreads), 0, stream, st, items, first, (double2*)aux);
      }
      break;
    case 3:
      if (count <= 0) return hipSuccess;
      {
        const auto kern = st.D <= 16 ? k_adj_rows<CT, 16> : k_adj_rows<CT, 32>;
        hipLaunchKernelGGL(kern, dim3(row_grid(st, count, blocks_per_slice)), dim3(256), 0, stream, st, items, first,
                           blocks_per_slice, (const double2*)aux);
      }
      break;
    case 6:  // lambda-bar of the other legs, both passes, over `count` items starting at `first`
      if (count <= 0) return hipSuccess;
      hipLaunchKernelGGL(k_adj_lbar, dim3(count * 2), dim3(256), 0, stream, st, items, first, 0);
      hipLaunchKernelGGL(k_adj_lbar, dim3(count * 2), dim3(256), 0, stream, st, items, first, 1);
      break;
    case 7:  // dL/dtheta per instance from the accumulators; count = number of RX chunks
      if (st.n_inst <= 0) return hipSuccess;
      hipLaunchKernelGGL(k_adj_theta, dim3(st.n_inst), dim3(256), 0, stream, st, count);
      break;
    case 4:  // readout seed over all vertices
      hipLaunchKernelGGL(k_adj_readout<CT>, dim3(st.NV), dim3(1024), 0, stream, st);
      break;
    case 5:  // RX adjoint over `count` chunks starting at `first`; aux = pre-RX site tensors
      if (count <= 0) return hipSuccess;
      hipLaunchKernelGGL(k_adj_rx<CT>, dim3(count), dim3(256), 0, stream, st, aux, first);
      break;
    default:
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_adjoint(int which, bool c128, const DevState& st, const int32_t* items, int first, int count,
                          int blocks_per_slice, const void* aux, hipStream_t stream) {
  return c128 ? adj_launch<double2>(which, st, items, first, count, blocks_per_slice, aux, stream)
              : adj_launch<float2>(which, st, items, first, count, blocks_per_slice, aux, stream);
}

hipError_t launch_checkpoint(const DevState& st, const void* src, void* dst, int64_t bytes, int64_t slot_bytes,
                             hipStream_t stream) {
  const int64_t n32 = bytes / 4;
  const int64_t blocks64 = (n32 + 255) / 256;
  const int blocks = (int)(blocks64 < 4096 ? (blocks64 > 0 ? blocks64 : 1) : 4096);
  hipLaunchKernelGGL(k_checkpoint, dim3(blocks), dim3(256), 0, stream, (const uint32_t*)src, (uint32_t*)dst, n32,
                     slot_bytes / 4, st.step_ctr, st.max_steps);
  return hipGetLastError();
}

hipError_t launch_mean_z(const DevState& st, int row, hipStream_t stream) {
  if (st.n_inst <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_mean_z, dim3(st.n_inst), dim3(256), 0, stream, st, row);
  return hipGetLastError();
}

hipError_t launch_seed_mean(const DevState& st, hipStream_t stream) {
  if (st.NV <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_seed_mean, dim3((st.NV + 255) / 256), dim3(256), 0, stream, st);
  return hipGetLastError();
}

hipError_t launch_fill_d(double* p, int64_t n, hipStream_t stream) {
  const int64_t blocks64 = (n + 255) / 256;
  const int blocks = (int)(blocks64 < 4096 ? (blocks64 > 0 ? blocks64 : 1) : 4096);
  hipLaunchKernelGGL(k_fill_d, dim3(blocks), dim3(256), 0, stream, p, n);
  return hipGetLastError();
}

}  // namespace gpeps
