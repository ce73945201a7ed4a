// Belief propagation (BP) on the norm network <psi|psi> of the graph PEPS, for gfx950.
//
// The simple update's lambda environment is the fixed point of BP on the norm network, and BP
// gauging after each step does not improve on it (Results, discussion of Fig. 3(a)).  These
// kernels run BP on the current state without changing it, which measures how far the
// simple-update gauge is from that fixed point:
//   * site tensors in the symmetric gauge A_v = Gamma_v sqrt(lambda_e) on every leg e;
//   * one message per directed edge, a D x D complex float64 matrix over the ket and bra copies
//     of the bond index (zero outside the active chi_e x chi_e block), starting at
//     identity / chi_e; slot 2 e + d holds the message from end d of edge e into end 1 - d;
//   * k_bp_update: one parallel iteration, one workgroup per directed edge and block of 16 rows:
//       m[a, a'] = sum_{s, b, b', c, c'} A[s, a, b, c] conj(A[s, a', b', c']) M1[b, b'] M2[c, c']
//     (a on the edge's leg, b and c on the sender's other legs, M1 and M2 the messages into the
//     sender along them);
//     divided by its trace (above D = 16 in a launch of its own, k_bp_norm); with the last one the
//     largest Frobenius
//     change of a message goes to the residual word;
//   * k_bp_readout: one workgroup per qubit and block of 16 rows, rho[s, s] with every leg closed
//     by its incoming message; k_bp_z: <Z> = (rho_00 - rho_11) / (rho_00 + rho_11).
// The work is 48 D^4 operations per directed edge of a sender with three legs, three dense
// products per physical slice, all in float64 on the matrix cores (bp_block below).

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>

#include "gpeps_device.h"
#include "gpeps_internal.h"

namespace gpeps {

namespace {

// N: bound on D that sizes a kernel (8, 16 or 32).  Eight waves a workgroup from D = 9 on; four below,
// where a wave already has two products of a phase at most and small workgroups share a CU.
template <int N> constexpr int bp_threads() { return N == 8 ? 256 : 512; }
template <int N> constexpr int bp_tiles() { return N == 32 ? 2 : 1; }  // 16-column tiles of a bond
typedef double bp_d4 __attribute__((ext_vector_type(4)));

// Geometry of one site tensor as seen by a BP contraction: leg 0 is `a`, legs 1 and 2 are b, c.
struct BpSite {
  int64_t base;     // element offset of the tensor
  int64_t pstride;  // stride of the physical index
  int32_t st[3];    // element strides of a, b, c (0 when absent)
  int32_t dim[3];   // active dimensions (1 when absent)
  int32_t edge[3];  // global edge ids (-1 when absent)
  int32_t in[3];    // message slots into this site along a, b, c (-1 when absent)
};

__device__ __forceinline__ int side_of(const DevState& st, int e, int64_t goff) {
  return st.edges[e].side[0].goff == goff ? 0 : 1;
}

// Entry [k][kp] of a message weighted by sqrt(lambda) of its leg on both indices: zero past the
// active n x n block; an absent leg (M null, n = 1) has the message [[1]].
template <int N>
__device__ __forceinline__ double2 bp_wmsg(const double2* M, int D, int n, const double (&sl)[N], int k, int kp) {
  if (k >= n || kp >= n) return make_double2(0.0, 0.0);
  if (!M) return make_double2(1.0, 0.0);
  return cscale(M[k * D + kp], sl[k] * sl[kp]);
}

// The contraction of one physical slice for the 16 rows a0 .. a0 + 15 of the message:
//   m[a][a'] += sum_{b, b', c, c'} G[s, a, b, c] conj(G[s, a', b', c']) W1[b][b'] W2[c][c']
// with the raw site tensor G and the messages W weighted by sqrt(lambda) on both indices (the
// weights of leg a are applied by the caller), as three products on v_mfma_f64_16x16x4f64 (lane
// l supplies A[l % 16][l / 16] and B[l / 16][l % 16] of a k step of 4 and receives
// D[l / 16 + 4 r][l % 16]; a complex product is four real ones).  For every tile of 16 columns c':
//   X[a][c'] of every b  = sum_c G[a][b][c] W2[c][c']   (one product per b, the waves in turn; to LDS)
//   Y[b'][a] of every c' = sum_b W1[b][b'] X[a][b][c']  (one product per c', the waves in turn)
//   m[a][a']            += sum_b' Y[b'][a] conj(G[a'][b'][c'])
// Y is formed with b' on the rows, so the register that receives Y[4 r + l / 16][l % 16] is the
// operand of k step r of the last product as it stands: only X goes through LDS (beside W1, which
// the caller has put there, [b][b'] with row stride N + 1).  Lane l ends with m[a0 + l / 16 + 4 r][16 t + l % 16], this wave's share, in (mr[t][r], mi[t][r]).
// Bound by the FP64 matrix cores at D = 32, where one workgroup fills a CU's LDS (149 KB) with two
// waves per SIMD; at D <= 16 by the latency of the phases.  Every wave of the workgroup calls this.
template <typename CT, int N, int NB = bp_tiles<N>()>
__device__ __forceinline__ void bp_block(const CT* __restrict__ gam, const BpSite& g, const double2* W1,
                                         const double2* __restrict__ M2, int D, const double (&sl)[3][N], int a0,
                                         int s, double2* Xs, bp_d4 (&mr)[NB], bp_d4 (&mi)[NB]) {
  constexpr int kWaves = bp_threads<N>() / 64;
  constexpr int KS = N / 4;               // k steps of 4 over a bond
  constexpr int R4 = N < 16 ? N / 4 : 4;  // and over a tile of 16
  constexpr int PF = sizeof(CT) == sizeof(float2) ? NB : 1;
  constexpr int CS = N * 16 + 1;    // stride of c' in Xs[c'][b][a] (odd: writes free of bank conflicts)
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, li = l & 15, lk = l >> 4;
  const int na = g.dim[0], nb = g.dim[1], nc = g.dim[2];
  const CT* const gs = gam + g.base + s * g.pstride;
  // loads are at a valid offset in any case and zeroed when they are used: a choice between the
  // element and a zero becomes a flat load through the stack, and a select at the load waits for it
  auto at = [&](bool v, int off) -> CT { return gs[v ? off : 0]; };
  auto pick = [](bool v, const CT& x) { return v ? to_d2(x) : make_double2(0.0, 0.0); };
  const int ta = g.st[0], tb = g.st[1], tc = g.st[2];  // (a tensor has at most 2^16 elements)
  const int kb = (nb + 3) >> 2, kc = (nc + 3) >> 2;
  const bool av = a0 + li < na;
  const int arow = (av ? a0 + li : 0) * ta;
  for (int j = 0; 16 * j < nc; ++j) {
    double2 w2[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) w2[ks] = bp_wmsg<N>(M2, D, nc, sl[2], 4 * ks + lk, 16 * j + li);
    // X of this wave's b; the next b's elements are in flight while the products run
    CT nx[KS];
    auto fetch = [&](int b) {
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int c = 4 * ks + lk;
        nx[ks] = at(av && c < nc, arow + b * tb + c * tc);
      }
    };
    if (wv < nb) fetch(wv);
    for (int b = wv; b < nb; b += kWaves) {
      CT x[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) x[ks] = nx[ks];
      if (b + kWaves < nb) fetch(b + kWaves);
      bp_d4 xr = {0.0, 0.0, 0.0, 0.0}, xi = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks < kc) {
          const double2 a = pick(av && 4 * ks + lk < nc, x[ks]);
          xr = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, w2[ks].x, xr, 0, 0, 0);
          xi = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, w2[ks].y, xi, 0, 0, 0);
          xr = __builtin_amdgcn_mfma_f64_16x16x4f64(-a.y, w2[ks].y, xr, 0, 0, 0);
          xi = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, w2[ks].x, xi, 0, 0, 0);
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (N >= 16 || li < N) Xs[li * CS + b * 16 + lk + 4 * r] = make_double2(xr[r], xi[r]);
    }
    __syncthreads();
    const int ncp = min(16, nc - 16 * j);
    for (int cp = wv; cp < ncp; cp += kWaves) {
      // the elements of the last product (its first PF column tiles) ahead: they arrive while Y is
      // formed; complex128 has registers for one tile in flight
      CT ga[PF][NB][R4];
      auto fetch_last = [&](int ta2, CT (&x)[NB][R4]) {
#pragma unroll
        for (int t = 0; t < NB; ++t)
#pragma unroll
          for (int r = 0; r < R4; ++r) {
            const int a2 = 16 * ta2 + li, b2 = 16 * t + 4 * r + lk;
            x[t][r] = at(a2 < na && b2 < nb, a2 * ta + b2 * tb + (16 * j + cp) * tc);
          }
      };
#pragma unroll
      for (int at = 0; at < PF; ++at) fetch_last(at, ga[at]);
      bp_d4 yr[NB], yi[NB];
#pragma unroll
      for (int t = 0; t < NB; ++t) {
        yr[t] = (bp_d4){0.0, 0.0, 0.0, 0.0};
        yi[t] = (bp_d4){0.0, 0.0, 0.0, 0.0};
      }
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks < kb) {
          const int b = 4 * ks + lk;
          const double2 x = b < nb ? Xs[cp * CS + b * 16 + li] : make_double2(0.0, 0.0);
#pragma unroll
          for (int t = 0; t < NB; ++t) {
            const double2 w = N >= 16 || li < N ? W1[b * (N + 1) + 16 * t + li] : make_double2(0.0, 0.0);
            yr[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(w.x, x.x, yr[t], 0, 0, 0);
            yi[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(w.x, x.y, yi[t], 0, 0, 0);
            yr[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(-w.y, x.y, yr[t], 0, 0, 0);
            yi[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(w.y, x.x, yi[t], 0, 0, 0);
          }
        }
      }
#pragma unroll
      for (int at = 0; at < NB; ++at) {
        if (16 * at < na) {
          if (at >= PF) fetch_last(at, ga[at % PF]);
#pragma unroll
          for (int t = 0; t < NB; ++t)
#pragma unroll
            for (int r = 0; r < R4; ++r) {
              if (16 * t + 4 * r < nb) {
                const double2 c = pick(16 * at + li < na && 16 * t + 4 * r + lk < nb, ga[at % PF][t][r]);  // conjugated below
                mr[at] = __builtin_amdgcn_mfma_f64_16x16x4f64(yr[t][r], c.x, mr[at], 0, 0, 0);
                mi[at] = __builtin_amdgcn_mfma_f64_16x16x4f64(yi[t][r], c.x, mi[at], 0, 0, 0);
                mr[at] = __builtin_amdgcn_mfma_f64_16x16x4f64(yi[t][r], c.y, mr[at], 0, 0, 0);
                mi[at] = __builtin_amdgcn_mfma_f64_16x16x4f64(-yr[t][r], c.y, mi[at], 0, 0, 0);
              }
            }
        }
      }
    }
    __syncthreads();  // Xs is overwritten by the next tile, slice or reduction
  }
}

// LDS of bp_block; the per-wave sums of bp_reduce use the same memory.
template <int N> constexpr int bp_lds() {
  constexpr int x = (N < 16 ? N : 16) * (N * 16 + 1), y = bp_threads<N>() * bp_tiles<N>() * 4;
  return x > y ? x : y;
}

// Adds the waves' shares of m in a fixed order: entry q < NB * 256 of the 16 x 16 NB block sits at
// register slot q / 64 = 4 t + r and lane q % 64.  put(i, j, v) receives row i (0 .. 15) and column j
// (0 .. 16 NB - 1); a thread gets at most one entry.
template <int N, class F, int NB = bp_tiles<N>()>
__device__ __forceinline__ void bp_reduce(double2* lds, const bp_d4 (&mr)[NB], const bp_d4 (&mi)[NB], F put) {
  constexpr int kWaves = bp_threads<N>() / 64;
  static_assert(NB * 256 <= bp_threads<N>(), "one entry a thread");
  const int l = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int t = 0; t < NB; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) lds[((wv * NB + t) * 4 + r) * 64 + l] = make_double2(mr[t][r], mi[t][r]);
  __syncthreads();
  const int q = threadIdx.x;
  if (q < NB * 256) {
    double2 v = lds[q];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v = cadd(v, lds[w * NB * 256 + q]);
    const int t = q >> 8, r = (q >> 6) & 3, ll = q & 63;
    put((ll >> 4) + 4 * r, 16 * t + (ll & 15), v);
  }
}

// sqrt(lambda) of the three legs (1 for an absent one), then the weighted message along leg b.
template <int N>
__device__ __forceinline__ void bp_weights(const DevState& st, const BpSite& g, const double2* M1,
                                           double (&sl)[3][N], double2* W1) {
#pragma unroll
  for (int l = 0; l < 3; ++l)
    if (threadIdx.x < N) {
      const int k = threadIdx.x;
      sl[l][k] = g.edge[l] >= 0 ? (k < st.D ? sqrt(st.lam[(int64_t)g.edge[l] * st.D + k]) : 0.0) : 1.0;
    }
  __syncthreads();
  for (int i = threadIdx.x; i < N * N; i += bp_threads<N>()) {
    const int k = i / N, kp = i - (i / N) * N;
    W1[k * (N + 1) + kp] = bp_wmsg<N>(M1, st.D, g.dim[1], sl[1], k, kp);
  }
  __syncthreads();
}

// A non-negative residual folded into the residual word (such doubles order like their bit patterns).
__device__ __forceinline__ void bp_record(const DevState& st, double dev2) {
  const double r = sqrt(dev2);
  atomicMax(st.bp_res, (unsigned long long)__double_as_longlong(isfinite(r) ? r : 0.0));
}

}  // namespace

// Identity / chi_e on the active block of every message of buffer 0; clears the residual word.
__global__ void k_bp_init(DevState st) {
  const int D = st.D;
  const int slot = blockIdx.x;
  const int chi = st.chi[slot >> 1];
  double2* m = st.bp_msg + (int64_t)slot * D * D;
  for (int i = threadIdx.x; i < D * D; i += blockDim.x) {
    const int r = i / D, c = i - (i / D) * D;
    m[i] = make_double2(r == c && r < chi ? 1.0 / chi : 0.0, 0.0);
  }
  if (slot == 0 && threadIdx.x == 0) *st.bp_res = 0ull;
}

// One parallel BP iteration: messages of buffer `src` -> buffer 1 - src.  Up to D = 16 a workgroup holds
// its whole message and divides it by its trace; above, that is left to k_bp_norm.
// Small bonds are bound by the launch: ten iterations and the readout of the 127-qubit graph take
// 172 us at D = 2 in complex128 (226 with k_bp_norm at every D, 181 before the matrix cores), and
// sixteen such instances at D = 3 470 us with kernels sized for D <= 8 (1129 with those for 16, 580).
// Measured at D = 32 on the 288 directed edges of the 127-qubit graph: 180 us (5.4 GFLOP, 30 TFLOP/s)
// with the senders of three legs first (bp_order), 307 us in edge order (some CUs got two of their
// 150 us workgroups), 3860 us as vector dot products with one workgroup per directed edge.
template <typename CT, int N>
__global__ __launch_bounds__(bp_threads<N>()) void k_bp_update(DevState st, int src, int record) {
  constexpr int NB = bp_tiles<N>();
  __shared__ double2 Xs[bp_lds<N>()];
  __shared__ double2 W1[N * (N + 1)];
  __shared__ double sl[3][N];
  __shared__ double red[8];
  const int D = st.D;
  const int nab = (D + 15) >> 4;  // blocks of 16 rows
  const int ord = blockIdx.x / nab, a0 = 16 * (blockIdx.x - ord * nab);
  const int slot = st.bp_order[ord];
  const int e = slot >> 1, d = slot & 1;
  const SideInfo& S = st.edges[e].side[d];
  BpSite g;
  g.base = S.goff;
  g.pstride = S.pstride;
  g.st[0] = S.sq;
  g.dim[0] = st.chi[e];
  g.edge[0] = e;
  g.in[0] = -1;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int f = S.oth[k];
    g.edge[1 + k] = f;
    g.st[1 + k] = f >= 0 ? S.so[k] : 0;
    g.dim[1 + k] = f >= 0 ? st.chi[f] : 1;
    g.in[1 + k] = f >= 0 ? 2 * f + (1 - side_of(st, f, S.goff)) : -1;
  }
  const int64_t nmsg = (int64_t)2 * st.NE * D * D;
  const double2* msg = st.bp_msg + (src ? nmsg : 0);
  double2* out = st.bp_msg + (src ? 0 : nmsg) + (int64_t)slot * D * D;
  const double2* M1 = g.in[1] >= 0 ? msg + (int64_t)g.in[1] * D * D : nullptr;
  const double2* M2 = g.in[2] >= 0 ? msg + (int64_t)g.in[2] * D * D : nullptr;
  bp_weights<N>(st, g, M1, sl, W1);
  bp_d4 mr[NB], mi[NB];
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    mr[t] = (bp_d4){0.0, 0.0, 0.0, 0.0};
    mi[t] = (bp_d4){0.0, 0.0, 0.0, 0.0};
  }
  if (a0 < g.dim[0]) {
    for (int s = 0; s < 2; ++s)
      bp_block<CT, N>(reinterpret_cast<const CT*>(st.gamma), g, W1, M2, D, sl, a0, s, Xs, mr, mi);
  }
  int at = -1;  // this thread's entry of the message
  double2 mine = make_double2(0.0, 0.0);
  bool diag = false;
  bp_reduce<N>(Xs, mr, mi, [&](int i, int j, double2 v) {
    const int a = a0 + i;
    if (a < D && j < D) {
      at = a * D + j;
      diag = a == j;
      if (a < g.dim[0] && j < g.dim[0]) mine = cscale(v, sl[0][a] * sl[0][j]);
    }
  });
  if constexpr (N == 32) {
    if (at >= 0) out[at] = mine;
  } else {
    const int tid = threadIdx.x, l = tid & 63, wv = tid >> 6;  // the entries sit in the first four waves
    const double t = group_sum(diag ? mine.x : 0.0, 64);
    if (l == 0 && wv < 4) red[wv] = t;
    __syncthreads();
    const double tr = (red[0] + red[1]) + (red[2] + red[3]);
    const bool good = isfinite(tr) && tr > 0.0;
    const double2 v = cscale(mine, good ? 1.0 / tr : 0.0);
    if (at >= 0) out[at] = v;
    if (record) {
      const double dv = group_sum(at >= 0 ? cabs2(csub(v, msg[(int64_t)slot * D * D + at])) : 0.0, 64);
      if (l == 0 && wv < 4) red[4 + wv] = dv;
      __syncthreads();
      if (tid == 0) bp_record(st, (red[4] + red[5]) + (red[6] + red[7]));
    }
    if (tid == 0 && !good) flag_status(st.status, kStatusNonFinite);
  }
}

// Above D = 16: the new messages (buffer 1 - src) divided by their traces; with `record` the largest Frobenius
// change against buffer src is folded into the residual word.
__global__ __launch_bounds__(256) void k_bp_norm(DevState st, int src, int record) {
  __shared__ double red[4];
  const int D = st.D, slot = blockIdx.x, tid = threadIdx.x;
  const int64_t nmsg = (int64_t)2 * st.NE * D * D;
  const double2* old = st.bp_msg + (src ? nmsg : 0) + (int64_t)slot * D * D;
  double2* out = st.bp_msg + (src ? 0 : nmsg) + (int64_t)slot * D * D;
  const int l = tid & 63;
  // every wave forms the trace by itself (the same sum in each)
  const double tr = group_sum(l < D ? out[l * D + l].x : 0.0, 64);
  const bool good = isfinite(tr) && tr > 0.0;
  const double inv = good ? 1.0 / tr : 0.0;
  __syncthreads();  // the diagonal has been read by every wave
  double dev = 0.0;
  for (int i = tid; i < D * D; i += 256) {
    const double2 v = cscale(out[i], inv);
    if (record) dev += cabs2(csub(v, old[i]));
    out[i] = v;
  }
  if (record) {
    dev = group_sum(dev, 64);
    if (l == 0) red[tid >> 6] = dev;
    __syncthreads();
  }
  if (tid == 0) {
    if (!good) flag_status(st.status, kStatusNonFinite);
    if (record) bp_record(st, (red[0] + red[1]) + (red[2] + red[3]));
  }
}

// The directed edge out of vertex v along its first leg: where the readout keeps v's partial sums.
__device__ __forceinline__ int bp_vertex_slot(const DevState& st, const VertexInfo& V) {
  return 2 * V.leg[0] + side_of(st, V.leg[0], V.goff);
}

// BP readout from the messages of buffer `buf`: rho[s, s] of the rows a0 .. a0 + 15 of the first leg
// of a qubit, into the other buffer (free after the last iteration): two doubles per block of rows,
// at the slot of the qubit's first leg.  Qubits without legs are left to k_bp_z.
template <typename CT, int N>
__global__ __launch_bounds__(bp_threads<N>()) void k_bp_readout(DevState st, int buf) {
  constexpr int NB = bp_tiles<N>();
  constexpr int kWaves = bp_threads<N>() / 64;
  __shared__ double2 Xs[bp_lds<N>()];
  __shared__ double2 W1[N * (N + 1)];
  __shared__ double sl[3][N];
  __shared__ double red[kWaves];
  const int D = st.D;
  const int nab = (D + 15) >> 4;
  const int v = blockIdx.x / nab, ab = blockIdx.x - v * nab, a0 = 16 * ab;
  const VertexInfo& V = st.verts[v];
  if (V.deg == 0) return;
  BpSite g;
  g.base = V.goff;
  int64_t ps = 1;
  for (int l = 0; l < V.deg; ++l) ps *= D;
  g.pstride = ps;
  int64_t stride = ps;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const int f = l < V.deg ? V.leg[l] : -1;
    g.edge[l] = f;
    if (f >= 0) stride /= D;
    g.st[l] = f >= 0 ? (int32_t)stride : 0;
    g.dim[l] = f >= 0 ? st.chi[f] : 1;
    g.in[l] = f >= 0 ? 2 * f + (1 - side_of(st, f, V.goff)) : -1;
  }
  const int64_t nmsg = (int64_t)2 * st.NE * D * D;
  const double2* msg = st.bp_msg + (buf ? nmsg : 0);
  double* part = reinterpret_cast<double*>(st.bp_msg + (buf ? 0 : nmsg) + (int64_t)bp_vertex_slot(st, V) * D * D) + 2 * ab;
  const double2* M0 = msg + (int64_t)g.in[0] * D * D;
  const double2* M1 = g.in[1] >= 0 ? msg + (int64_t)g.in[1] * D * D : nullptr;
  const double2* M2 = g.in[2] >= 0 ? msg + (int64_t)g.in[2] * D * D : nullptr;
  bp_weights<N>(st, g, M1, sl, W1);
  for (int s = 0; s < 2; ++s) {
    bp_d4 mr[NB], mi[NB];
#pragma unroll
    for (int t = 0; t < NB; ++t) {
      mr[t] = (bp_d4){0.0, 0.0, 0.0, 0.0};
      mi[t] = (bp_d4){0.0, 0.0, 0.0, 0.0};
    }
    if (a0 < g.dim[0]) bp_block<CT, N>(reinterpret_cast<const CT*>(st.gamma), g, W1, M2, D, sl, a0, s, Xs, mr, mi);
    // rho[s, s] = sum_{a, a'} M0[a][a'] m[a][a'] (real: M0 and m are Hermitian)
    double acc = 0.0;
    bp_reduce<N>(Xs, mr, mi, [&](int i, int j, double2 m) {
      const int a = a0 + i;
      if (a < g.dim[0] && j < g.dim[0]) acc += cmul(M0[a * D + j], m).x * (sl[0][a] * sl[0][j]);
    });
    acc = group_sum(acc, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double r = 0.0;
      for (int w = 0; w < kWaves; ++w) r += red[w];
      part[s] = r;
    }
    __syncthreads();
  }
}

// <Z> of every qubit from the partial sums of k_bp_readout (a qubit without legs from its tensor).
template <typename CT>
__global__ __launch_bounds__(256) void k_bp_z(DevState st, int buf) {
  const int v = blockIdx.x * 256 + threadIdx.x;
  if (v >= st.NV) return;
  const VertexInfo& V = st.verts[v];
  const int D = st.D, nab = (D + 15) >> 4;
  double r0 = 0.0, r1 = 0.0;
  if (V.deg == 0) {
    const CT* gam = reinterpret_cast<const CT*>(st.gamma) + V.goff;
    r0 = cabs2(to_d2(gam[0]));
    r1 = cabs2(to_d2(gam[1]));
  } else {
    const int64_t nmsg = (int64_t)2 * st.NE * D * D;
    const double* part = reinterpret_cast<const double*>(st.bp_msg + (buf ? 0 : nmsg) + (int64_t)bp_vertex_slot(st, V) * D * D);
    for (int b = 0; b < nab; ++b) {
      r0 += part[2 * b];
      r1 += part[2 * b + 1];
    }
  }
  const double zv = (r0 - r1) / (r0 + r1);
  if (!isfinite(zv)) flag_status(st.status, kStatusNonFinite);
  st.z[v] = zv;
}

template <typename CT, int N>
void launch_bp_t(const DevState& st, int iters, hipStream_t stream) {
  const int slots = 2 * st.NE, nab = (st.D + 15) / 16;
  constexpr int threads = bp_threads<N>();
  if (slots > 0) {
    hipLaunchKernelGGL(k_bp_init, dim3(slots), dim3(256), 0, stream, st);
    for (int it = 0; it < iters; ++it) {
      const int last = it == iters - 1;
      hipLaunchKernelGGL((k_bp_update<CT, N>), dim3(slots * nab), dim3(threads), 0, stream, st, it & 1, last);
      if (N == 32) hipLaunchKernelGGL(k_bp_norm, dim3(slots), dim3(256), 0, stream, st, it & 1, last);
    }
  }
  if (st.NV > 0) {
    if (slots > 0) hipLaunchKernelGGL((k_bp_readout<CT, N>), dim3(st.NV * nab), dim3(threads), 0, stream, st, iters & 1);
    hipLaunchKernelGGL(k_bp_z<CT>, dim3((st.NV + 255) / 256), dim3(256), 0, stream, st, iters & 1);
  }
}

// ------------------------------------------------------------------ device-resident BP scratch
//
// The messages and the residual word of gpeps_bp_expect_z_noalloc live in this array instead of
// the caller's workspace, for callers that cannot allocate.  Every GPU the library runs on holds
// its own copy until the process ends; host code never uses the name itself (a host-side stand-in)
// but the device address returned by hipGetSymbolAddress, recorded once per device.
static __device__ __align__(256) unsigned char scratch[kBpScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
hipError_t g_scratch_err[kMaxDevices] = {};
bool g_scratch_done[kMaxDevices] = {};
}  // namespace

// Device address of `scratch` on the current device, looked up on the first call for that
// device.  Returns the lookup's status (kept per device) and writes the address to *ptr.
hipError_t bp_scratch_address(void** ptr) {
  *ptr = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_done[dev]) {
    void* p = nullptr;
    g_scratch_err[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    g_scratch_ptr[dev] = g_scratch_err[dev] == hipSuccess ? p : nullptr;
    g_scratch_done[dev] = true;
  }
  *ptr = g_scratch_ptr[dev];
  return g_scratch_err[dev];
}

hipError_t launch_bp(bool c128, const DevState& st, int iters, hipStream_t stream) {
  if (st.D > kMaxD) return hipErrorInvalidValue;
  if (st.D <= 8) {
    if (c128) launch_bp_t<double2, 8>(st, iters, stream);
    else launch_bp_t<float2, 8>(st, iters, stream);
  } else if (st.D <= 16) {
    if (c128) launch_bp_t<double2, 16>(st, iters, stream);
    else launch_bp_t<float2, 16>(st, iters, stream);
  } else {
    if (c128) launch_bp_t<double2, 32>(st, iters, stream);
    else launch_bp_t<float2, 32>(st, iters, stream);
  }
  return hipGetLastError();
}

}  // namespace gpeps
