// am_setup.hip -- one-time FP64 construction of the constant operators of the
// batched AM iteration (Sec. III-A eqs. over_2/over_3; Sec. IV: F^T F is
// formed once), on the GPU.
//
// The Bernstein basis P (eq. param) is factored P = U R with U orthonormal on
// the time grid.  The iteration runs on z = R c: x = U z, xdot = V z,
// xddot = W z with V = Pdot R^-1, W = Pddot R^-1.  In these coordinates the
// Gram matrix of the position rows is the identity, so the xi1 KKT matrix is
// well conditioned and its FP32 application does not amplify rounding the way
// the Bernstein-coordinate inverse does.  The KKT matrices are assembled in z
// coordinates and inverted by Gauss-Jordan elimination with partial pivoting.
//
// A set-up is a chain of small dependent steps, so latency bounds it: the
// first kernel is one workgroup that holds every matrix in LDS (about 100 KB)
// and runs each step on as many lanes as it has entries, the second spreads
// what only depends on its results (products for the iteration, Bernstein
// inverses, typed copies) over the GPU.  A first form in one workgroup with
// its matrices in global memory (serial pivot searches, one block-wide
// reduction per Gram-Schmidt coefficient) took 556 us; these take 59 + 13 us
// (q = 100, nv = 11, set-ups repeated: basis 8, QR 17, elimination 25, Gram
// matrices 2 us; as the only one of a process the second kernel, whose
// unrolled jobs hold 368 bytes of scratch a lane, took 14 to 75 us).
#include <hip/hip_runtime.h>

#include "am_device.h"
#include "am_internal.h"

namespace amk {
namespace {

constexpr int kSetupThreads = 1024;
constexpr int kPackBlocks = 6, kPackThreads = 256;

struct SetupArgs {
  int q, m, n, flags, f64;
  double tf, rho;
  double r[AM_MAX_CIRCLES];
  Consts c;
};

// LDS of the first kernel, in doubles.
template <int NV>
struct SetupLds {
  static constexpr int N1 = 2 * NV + 6, N2 = NV + 6;
  int P, Pd, Pdd, U, V, W, R, Rinv, G, bin, vcol, dj, A1, A2, total;
  __host__ __device__ explicit SetupLds(int q) {
    int o = 0;
    P = o; o += q * NV;
    Pd = o; o += q * NV;
    Pdd = o; o += q * NV;
    U = o; o += q * NV;
    V = o; o += q * NV;
    W = o; o += q * NV;
    R = o; o += NV * NV;
    Rinv = o; o += NV * NV;
    G = o; o += 3 * NV * NV;
    bin = o; o += 3 * NV;
    vcol = o; o += 2 * AM_MAX_Q;
    dj = o; o += NV;
    A1 = o; o += 2 * N1 * (2 * N1 + 1);   // augmented [N][2N + 1], two buffers
    A2 = o; o += 2 * N2 * (2 * N2 + 1);
    total = o;
  }
};

// Bernstein polynomial B_{deg,i}(tau) with the binomials of `deg` in `bin`;
// zero outside 0 <= i <= deg.
__device__ __noinline__ double bernstein(const double *bin, int deg, int i, double tau) {
  if (i < 0 || i > deg) return 0.0;
  double v = bin[i];
  for (int k = 0; k < i; ++k) v *= tau;
  for (int k = 0; k < deg - i; ++k) v *= (1.0 - tau);
  return v;
}

__device__ __forceinline__ double lane_sum(double v) {
  return wave_all(v, 0.0, [](double a, double b) { return a + b; });
}

// One column step of the Gauss-Jordan elimination of the augmented [N][2N]
// matrix (row stride 2N + 1: a column's entries lie in different LDS banks):
// reads `a`, writes `b`.  Every wavefront finds the pivot row by itself (the
// first row of largest magnitude at or below `col`), so a step needs one
// barrier.  Returns false if the pivot is at most `tol`.
template <int N, int THREADS>
__device__ bool gj_step(const double *__restrict__ a, double *__restrict__ b, int col, double tol, int tid) {
  constexpr int W2 = 2 * N, S = W2 + 1, E = (N * W2 + THREADS - 1) / THREADS;
  static_assert(N <= kWave, "one lane per row");
  const int lane = threadIdx.x & (kWave - 1);
  const bool row = lane >= col && lane < N;
  const double mine = row ? fabs(a[lane * S + col]) : -1.0;
  const double top = wave_all(mine, -1.0, [](double x, double y) { return fmax(x, y); });
  const unsigned long long at = __ballot(row && mine == top);
  if (!(top > tol) || at == 0) return false;   // (a NaN matrix has no pivot)
  const int p = __builtin_ctzll(at);
  double old[E], fac[E], prow[E];
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const int idx = tid + k * THREADS, r = idx / W2, c = idx % W2;
    if (idx < N * W2) {
      const int src = r == p ? col : r;   // rows p and col change places
      old[k] = a[src * S + c];
      fac[k] = a[src * S + col];
      prow[k] = a[p * S + c];
    }
  }
  const double inv = 1.0 / a[p * S + col];
#pragma unroll
  for (int k = 0; k < E; ++k) {
    const int idx = tid + k * THREADS, r = idx / W2, c = idx % W2;
    if (idx < N * W2) {
      const double pr = prow[k] * inv;
      b[r * S + c] = r == col ? pr : old[k] - fac[k] * pr;
    }
  }
  return true;
}

template <int NV>
__global__ __launch_bounds__(kSetupThreads) void setup_kernel(SetupArgs a) {
  constexpr int N = NV - 1, n2 = 2 * NV, N1 = n2 + 6, N2 = NV + 6, T = kSetupThreads;
  extern __shared__ __align__(16) double sm[];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int q = a.q;
  const Consts &c = a.c;
  const SetupLds<NV> L(q);
  double *P = sm + L.P, *Pd = sm + L.Pd, *Pdd = sm + L.Pdd, *U = sm + L.U, *V = sm + L.V, *W = sm + L.W;
  double *R = sm + L.R, *Rinv = sm + L.Rinv, *G = sm + L.G, *bin = sm + L.bin;

  // 1. Binomials C(deg, i) (built multiplicatively, exact), then the Bernstein
  //    basis and its time derivatives on t_k = k tf/(q-1).
  if (tid < 3 * NV) {
    const int deg = N - tid / NV, i = tid % NV;
    double v = 1.0;
    for (int k = 1; k <= i; ++k) v = v * double(deg - i + k) / double(k);
    bin[tid] = i <= deg ? v : 0.0;
    // (R is upper triangular)
  }
  for (int idx = tid; idx < NV * NV; idx += T) R[idx] = 0.0;
  __syncthreads();
  for (int idx = tid; idx < q * NV; idx += T) {
    const int t = idx / NV, i = idx % NV;
    const double tau = double(t) / double(q - 1);
    const double p = bernstein(bin, N, i, tau);
    const double pd = double(N) * (bernstein(bin + NV, N - 1, i - 1, tau) - bernstein(bin + NV, N - 1, i, tau)) / a.tf;
    const double pdd = double(N) * double(N - 1) *
                       (bernstein(bin + 2 * NV, N - 2, i - 2, tau) - 2.0 * bernstein(bin + 2 * NV, N - 2, i - 1, tau) +
                        bernstein(bin + 2 * NV, N - 2, i, tau)) / (a.tf * a.tf);
    P[idx] = p;
    Pd[idx] = pd;
    Pdd[idx] = pdd;
    c.P[idx] = p;
    c.Pd[idx] = pd;
    c.Pdd[idx] = pdd;
  }
  __syncthreads();
  // 2. Thin QR, P = U R, by Gram-Schmidt with one re-orthogonalisation pass:
  //    all coefficients of a pass at once, one per wavefront.  (Loops are kept
  //    rolled: unrolled code that runs once costs more in instruction
  //    fetches than it saves.)
  double *vcol = sm + L.vcol, *dj = sm + L.dj;
#pragma unroll 1
  for (int k = 0; k < NV; ++k) {
    double *vc = vcol + (k & 1) * AM_MAX_Q;
    double v = tid < q ? P[tid * NV + k] : 0.0;
    if (tid < AM_MAX_Q) vc[tid] = v;
    __syncthreads();
    if (k > 0) {
#pragma unroll 1
      for (int pass = 0; pass < 2; ++pass) {
#pragma unroll 1
        for (int j = wave; j < k; j += T / kWave) {
          const double x0 = lane < q ? U[lane * NV + j] : 0.0, x1 = lane + kWave < q ? U[(lane + kWave) * NV + j] : 0.0;
          const double d = lane_sum(x0 * vc[lane] + x1 * vc[lane + kWave]);
          if (lane == 0) {
            dj[j] = d;
            R[j * NV + k] += d;
          }
        }
        __syncthreads();
        if (tid < q) {
#pragma unroll
          for (int j = 0; j < NV - 1; ++j) {
            const int jj = j < k ? j : 0;   // (the loads of all columns are issued together)
            const double e = dj[jj] * U[tid * NV + jj];
            v -= j < k ? e : 0.0;
          }
          vc[tid] = v;
        }
        __syncthreads();
      }
    }
    const double w0 = vc[lane], w1 = vc[lane + kWave];
    const double nrm = sqrt(lane_sum(w0 * w0 + w1 * w1));
    if (tid < q) U[tid * NV + k] = v / nrm;
    if (tid == 0) R[k * NV + k] = nrm;
  }
  __syncthreads();
  // 3. R^-1 (upper triangular), a column per lane of one wavefront.
  if (tid < NV) {
    double x[NV];
#pragma unroll
    for (int i = NV - 1; i >= 0; --i) {
      double s = i == tid ? 1.0 : 0.0;
#pragma unroll
      for (int j = i + 1; j < NV; ++j) s -= R[i * NV + j] * x[j];
      x[i] = i > tid ? 0.0 : s / R[i * NV + i];
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) Rinv[i * NV + tid] = x[i];
  }
  __syncthreads();

  // 4. V = Pdot R^-1, W = Pddot R^-1.
  for (int idx = tid; idx < q * NV; idx += T) {
    const int t = idx / NV, k = idx % NV;
    double v = 0.0, w = 0.0;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      v += Pd[t * NV + j] * Rinv[j * NV + k];
      w += Pdd[t * NV + j] * Rinv[j * NV + k];
    }
    V[idx] = v;
    W[idx] = w;
    c.U[idx] = U[idx];
    c.V[idx] = v;
    c.W[idx] = w;
  }
  for (int idx = tid; idx < NV * NV; idx += T) {
    c.R[idx] = R[idx];
    c.Rinv[idx] = Rinv[idx];
  }
  __syncthreads();

  // 5. Gram matrices G_UU, G_VV, G_WW.
  for (int idx = tid; idx < 3 * NV * NV; idx += T) {
    const int which = idx / (NV * NV), e = idx % (NV * NV), i = e / NV, j = e % NV;
    const double *X = which == 0 ? U : (which == 1 ? V : W);
    double s = 0.0;
#pragma unroll 4
    for (int t = 0; t < q; ++t) s += X[t * NV + i] * X[t * NV + j];
    G[idx] = s;
    c.G[idx] = s;
  }
  __syncthreads();

  // 6. F^T F of one axis inside the two KKT matrices in z coordinates,
  //    augmented with the identity.  F rows: [V 0], [W 0], [U r_i U] per
  //    (i, j), [0 U]  (Sec. III-C).
  const double *GUU = G, *GVV = G + NV * NV, *GWW = G + 2 * NV * NV;
  double *A1 = sm + L.A1, *A2 = sm + L.A2;
  double sr = 0.0, sr2 = 0.0;
  for (int i = 0; i < a.m; ++i) { sr += a.r[i]; sr2 += a.r[i] * a.r[i]; }
  const double mn = double(a.m) * double(a.n), nsr = double(a.n) * sr, nsr2 = double(a.n) * sr2;
  const bool q_cs = !(a.flags & AM_Q_CS_ZERO);
  // boundary row e: U, V, W at t = 0 and t = q-1
  auto brow = [&](int e, int k) {
    const double *X = (e % 3 == 0) ? U : ((e % 3 == 1) ? V : W);
    return X[(e < 3 ? 0 : q - 1) * NV + k];
  };
  constexpr int S1 = 2 * N1 + 1, S2 = 2 * N2 + 1;
  for (int idx = tid; idx < N1 * 2 * N1; idx += T) {
    const int I = idx / (2 * N1), J = idx % (2 * N1);
    double v = 0.0;
    if (J >= N1) {
      v = J - N1 == I ? 1.0 : 0.0;
    } else if (I < n2 && J < n2) {
      const int i = I % NV, j = J % NV, bi = I / NV, bj = J / NV, e = i * NV + j;
      if (bi == 0 && bj == 0) v = GWW[e] + a.rho * (GVV[e] + GWW[e] + mn * GUU[e]);
      else if (bi == 1 && bj == 1) v = (q_cs ? GWW[e] : 0.0) + a.rho * ((nsr2 + 1.0) * GUU[e]);
      else v = a.rho * (nsr * GUU[e]);
    } else if (I < NV && J >= n2) {
      v = brow(J - n2, I);   // column block A'^T
    } else if (I >= n2 && J < NV) {
      v = brow(I - n2, J);   // row block A'
    }
    A1[I * S1 + J] = v;
  }
  // xi2: [W^T W + rho U^T U, A^T; A, 0]
  for (int idx = tid; idx < N2 * 2 * N2; idx += T) {
    const int I = idx / (2 * N2), J = idx % (2 * N2);
    double v = 0.0;
    if (J >= N2) v = J - N2 == I ? 1.0 : 0.0;
    else if (I < NV && J < NV) v = GWW[I * NV + J] + a.rho * GUU[I * NV + J];
    else if (I < NV) v = brow(J - NV, I);
    else if (J < NV) v = brow(I - NV, J);
    A2[I * S2 + J] = v;
  }
  for (int idx = tid; idx < 6 * NV; idx += T) c.Abc[idx] = brow(idx / NV, idx % NV);
  __syncthreads();

  // 7. Inverses, both matrices at once: half the wavefronts eliminate each.
  //    A pivot is too small below 1e-13 of the largest entry.
  const bool first = tid < T / 2;
  const int gtid = first ? tid : tid - T / 2;
  double *A = first ? A1 : A2;
  const int NN = first ? N1 : N2, SS = first ? S1 : S2;
  double big = 0.0;
  for (int idx = lane; idx < NN * NN; idx += kWave) big = fmax(big, fabs(A[(idx / NN) * SS + idx % NN]));
  big = wave_all(big, 0.0, [](double x, double y) { return fmax(x, y); });
  const double tol = 1e-13 * big;
  bool ok = big > 0.0;
  double *from = A, *to = A + NN * SS;
  for (int col = 0; col < N1; ++col) {
    if (ok && col < NN) {
      ok = first ? gj_step<N1, T / 2>(from, to, col, tol, gtid) : gj_step<N2, T / 2>(from, to, col, tol, gtid);
      double *s = from;
      from = to;
      to = s;
    }
    __syncthreads();
  }
  if (tid == 0) bin[0] = ok ? 0.0 : 1.0;
  if (tid == T / 2) bin[1] = ok ? 0.0 : 2.0;
  __syncthreads();
  const double status = bin[0] != 0.0 ? bin[0] : bin[1];
  if (tid == 0) c.status[0] = status;
  if (status != 0.0) return;

  // 8. The inverses, and the blocks used by the iteration: [z; mu] = Kinv
  //    [rhs; b].
  for (int idx = gtid; idx < NN * NN; idx += T / 2) {
    const int I = idx / NN, J = idx % NN;
    const double v = from[I * SS + NN + J];
    if (first) {
      c.K1[idx] = v;
      if (I < n2 && J < n2) c.M1[I * n2 + J] = v;
      else if (I < n2) c.H1[I * 6 + J - n2] = v;
    } else {
      c.K2[idx] = v;
      if (I < NV && J < NV) c.M2[I * NV + J] = v;
      else if (I < NV) c.H2[I * 6 + J - NV] = v;
    }
  }
}

// What only depends on the first kernel's results: one job per blockIdx.y,
// an entry per thread.
constexpr int kPackJobs = 15;

template <int NV, typename F>
__global__ __launch_bounds__(kPackThreads) void pack_kernel(SetupArgs a) {
  constexpr int n2 = 2 * NV, N1 = n2 + 6, N2 = NV + 6;
  const Consts &c = a.c;
  const int q = a.q, job = blockIdx.y, qn = q * NV;
  const int tid = blockIdx.x * kPackThreads + threadIdx.x, T = kPackBlocks * kPackThreads;
  const bool q_cs = !(a.flags & AM_Q_CS_ZERO);
  const double *GWW = c.G + 2 * NV * NV;
  // Bernstein-coordinate inverses T Kinv T^T with T = blkdiag(R^-1, ..., I6):
  // row I of T runs over the block of I (nz rows of such blocks)
  auto bernstein_inv = [&](const double *K, double *out, int n, int nz) {
    for (int idx = tid; idx < n * n; idx += T) {
      const int I = idx / n, J = idx % n;
      const bool bi = I < nz, bj = J < nz;
      const int k0 = bi ? I / NV * NV : I, l0 = bj ? J / NV * NV : J;
      double tj[NV], s = 0.0;
#pragma unroll
      for (int l = 0; l < NV; ++l) tj[l] = bj ? c.Rinv[(J % NV) * NV + l] : (l == 0 ? 1.0 : 0.0);
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        const double ti = bi ? c.Rinv[(I % NV) * NV + k] : (k == 0 ? 1.0 : 0.0);
        double row = 0.0;
#pragma unroll
        for (int l = 0; l < NV; ++l) row += K[(bi ? k0 + k : k0) * n + (bj ? l0 + l : l0)] * tj[l];
        s += ti * row;
      }
      out[idx] = s;
    }
  };
  // row t, column k of U~ = U M2^T: the heading step's rows premultiplied by M2
  auto ut_of = [&](int t, int k) {
    double v = 0.0;
#pragma unroll
    for (int j = 0; j < NV; ++j) v += c.U[t * NV + j] * c.M2[k * NV + j];
    return v;
  };
  const int hq = (q + 1) / 2;
  constexpr int NP = pad4(NV);
  if (job == 0) {
    bernstein_inv(c.K1, c.K1b_inv, N1, n2);
  } else if (job == 1) {
    bernstein_inv(c.K2, c.K2b_inv, N2, NV);
  } else if (job == 2) {
    for (int idx = tid; idx < qn; idx += T) c.UT[idx] = c.U[idx % q * NV + idx / q];
  } else if (job == 3) {
    // N = M1 Q with Q the smoothness block of the xi1 objective
    for (int idx = tid; idx < n2 * n2; idx += T) {
      const int I = idx / n2, J = idx % n2, bj = J / NV, j = J % NV;
      double v = 0.0;
      if (bj == 0 || q_cs)
#pragma unroll
        for (int k = 0; k < NV; ++k) v += c.M1[I * n2 + bj * NV + k] * GWW[k * NV + j];
      static_cast<F *>(c.tN)[J * n2 + I] = F(v);
    }
  } else if (job == 4) {
    // the fused kernel's lanes, typed constants (an element per thread)
    F *out = static_cast<F *>(c.lane_t);
    for (int idx = tid; idx < 4 * lane_t_quads(NV); idx += T) {
      const int e = idx % 4, lane = idx / 4 % kWave, piece = idx / (4 * kWave);
      const int I = lane < 4 * NV ? lane % n2 : 0, qb = I / NV, qi = I % NV;
      double v = 0.0;
      if (piece < 2 * NP) {
        const int half = piece / NP, which = piece % NP / (NP / 4), k = 4 * (piece % (NP / 4)) + e;
        // slot k holds row k xor lane within groups of 4
        const int r = (k & ~3) | ((k ^ lane) & 3), t = half * hq + lane;
        if (lane < hq && t < q && r < NV)
          v = which == 0 ? c.U[t * NV + r] : (which == 1 ? c.V[t * NV + r] : (which == 2 ? c.W[t * NV + r] : ut_of(t, r)));
      } else if (piece < lane_t_q(NV)) {
        const int J = 4 * (piece - lane_t_m1(NV)) + e;
        v = J < n2 ? c.M1[I * n2 + J] : 0.0;
      } else if (piece < lane_t_m2(NV)) {
        const int k = 4 * (piece - lane_t_q(NV)) + e;
        v = k < NV && (qb == 0 || q_cs) ? GWW[qi * NV + k] : 0.0;
      } else if (piece < lane_t_h2(NV)) {
        const int k = 4 * (piece - lane_t_m2(NV)) + e;
        v = k < NV && lane < NV ? c.M2[lane * NV + k] : 0.0;
      } else {
        const int k = 4 * (piece - lane_t_h2(NV)) + e;
        v = k < 6 && lane < NV ? c.H2[lane * 6 + k] : 0.0;
      }
      out[idx] = F(v);
    }
  } else if (job == 5) {
    // ... and the FP64 ones
    for (int idx = tid; idx < 2 * lane_d_pairs(NV); idx += T) {
      const int e = idx % 2, lane = idx / 2 % kWave, piece = idx / (2 * kWave);
      const int I = lane < 4 * NV ? lane % n2 : 0, kk = I % NV;
      double v = 0.0;
      if (piece < NP) {
        const int half = piece / (NP / 2), k = 2 * (piece % (NP / 2)) + e, t = half * hq + lane;
        if (lane < hq && t < q && k < NV) v = c.U[t * NV + k];
      } else if (piece < lane_d_piece(NV, 0)) {
        v = c.H1[I * 6 + 2 * (piece - lane_d_h1(NV)) + e];
      } else {
        const int which = (piece - lane_d_piece(NV, 0)) / (NP / 2);
        const int j = 2 * ((piece - lane_d_piece(NV, 0)) % (NP / 2)) + e;
        if (j < NV) {
          if (which == LD_Q) v = GWW[kk * NV + j];
          else if (which == LD_R_ROW) v = c.R[kk * NV + j];
          else if (which == LD_RINV_COL) v = c.Rinv[j * NV + kk];
          else if (which == LD_RINV_ROW) v = c.Rinv[kk * NV + j];
          else if (which == LD_R_COL) v = c.R[j * NV + kk];
          else v = lane < 12 ? c.Abc[(lane % 6) * NV + j] : 0.0;
        }
      }
      c.lane_d[idx] = v;
    }
  } else {
    // typed copies, time (or the output row) fastest: consecutive lanes of the
    // plain and residual kernels read consecutive elements
    const struct { const double *src; void *dst; int rows, cols; } copy[] = {
        {c.U, c.tU, q, NV}, {c.V, c.tV, q, NV}, {c.W, c.tW, q, NV}, {c.P, c.tP, q, NV}, {c.Pd, c.tPd, q, NV},
        {c.Pdd, c.tPdd, q, NV}, {c.M1, c.tM1, n2, n2}, {c.M2, c.tM2, 1, NV * NV}, {c.H2, c.tH2, 1, NV * 6}};
    static_assert(sizeof(copy) / sizeof(copy[0]) == kPackJobs - 6, "a job per copy");
#pragma unroll
    for (int k = 0; k < kPackJobs - 6; ++k)
      if (job == 6 + k)
        for (int i = tid; i < copy[k].rows * copy[k].cols; i += T)
          static_cast<F *>(copy[k].dst)[i] = F(copy[k].src[i % copy[k].rows * copy[k].cols + i / copy[k].rows]);
  }
}

template <int NV>
hipError_t run(const SetupArgs &a, hipStream_t st) {
  const size_t lds = size_t(SetupLds<NV>(a.q).total) * sizeof(double);
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&setup_kernel<NV>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((setup_kernel<NV>), dim3(1), dim3(kSetupThreads), lds, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (a.f64) hipLaunchKernelGGL((pack_kernel<NV, double>), dim3(kPackBlocks, kPackJobs), dim3(kPackThreads), 0, st, a);
  else hipLaunchKernelGGL((pack_kernel<NV, float>), dim3(kPackBlocks, kPackJobs), dim3(kPackThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_setup(const am_shape &s, const double *r, const Consts &c, bool f64, hipStream_t st) {
  SetupArgs a{};
  a.q = s.q; a.m = s.m; a.n = s.n_obs; a.flags = int(s.flags); a.f64 = f64 ? 1 : 0;
  a.tf = s.tf; a.rho = s.rho; a.c = c;
  for (int i = 0; i < s.m; ++i) a.r[i] = r[i];
  if (s.nv == 11) return run<11>(a, st);
  if (s.nv == 8) return run<8>(a, st);
  return hipErrorInvalidValue;
}

}  // namespace amk
