// HIP kernels (gfx950) of the time-fractional extra-stress update.
//
// The BDF2 and exponential steps run in blocks of six waves, one per tensor component: a wave streams
// its component's modes for a few points a lane, and the point's sums meet in LDS, where one lane per
// point solves the local system.  (The start-up, and BDF2 on whole 2-D FP64 grids, keep all components
// of a point in one lane.)
//   * BDF2 step (Sec. 4.1, eqs. BDF_Phi_k_n+1 and FP_discrete, pointwise in tensor
//     variables with the mode representation Y_k = X_k - c_k X):
//       P        = 2 X^n - X^{n-1}/2
//       h^_k     = 2 Y_k^n - Y_k^{n-1}/2,      Y_k^{n+1} = d_k h^_k + d_k c_k P
//       G        = sum_k eta_k h^_k + (sum_k eta_k c_k) P          (compensated, FP64)
//       [(b0 + eta/De) I - eta (kappa~ . + . kappa~^T)] X^{n+1} = P - A(G) + zeta^{n+1} S
//       tau^{n+1} = (gamma/dt) (eta X^{n+1} - G)
//     The modes are streamed once: two levels read, one level written into the slot of
//     the older level.  The c x c local system (c = 3 or 6) is solved in a lane's registers by
//     Gaussian elimination with partial pivoting.
//   * SDIRK2 start-up (first step from rest of the modes): two stage solves with the
//     same local matrix; the level-0 and level-1 modes are written.
//   * Exponential-mode step (an extension, not the paper's scheme): every mode solved
//     exactly for X linear on the step, one mode level updated in place, and the state
//     integrated as X^{n+1} - X^n = A(sum_k (X_k^{n+1} - X_k^n)) + zeta S.
// The mode loop is a pure stream (no MFMA: about one flop per byte); the loads of the next two to
// eight modes are in flight while one is worked on (stream_modes).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <type_traits>
#include <vector>

#include "tfs_device.h"
#include "tfs_internal.h"

namespace tfs {
namespace {
using namespace dev;

// One block folds the block partials in a fixed order.
__global__ __launch_bounds__(kBlock) void diag_finish_kernel(const double* __restrict__ part, int nparts,
                                                             double* __restrict__ diag) {
  DiagAcc a;
  for (int i = threadIdx.x; i < nparts; i += kBlock) {
    DiagAcc b;
    const double* q = part + (size_t)i * kNumDiag;
    b.mn1 = q[0]; b.mn2 = q[1]; b.mn3 = q[2]; b.mx = q[3]; b.sum = q[4]; b.cnt = q[5];
    diag_combine(a, b);
  }
  const DiagAcc r = block_reduce<kBlock / 64>(a);
  if (threadIdx.x == 0) {
    diag[0] = r.mn1; diag[1] = r.mn2; diag[2] = r.mn3; diag[3] = r.mx; diag[4] = r.sum; diag[5] = r.cnt;
  }
}

// ------------------------------------------------------------------ BDF2 step
// Spatial form (eps Laplace where it is diagonal): each point is one coefficient of a
// field in a basis of Laplace eigenfunctions.  -eps Laplace acts on it as the extra
// relaxation rate eps |xi|^2, and only the constant function's coefficient carries the
// mass-mode source (the mass mode is the constant 1).
struct SpatialArgs {
  const double* rate;   // [stride] extra relaxation rate per point, or null (none)
  int64_t src;          // the point with the mass-mode source, or -1 (every point)
};

// The extra rate and the source weight (1 or 0) of the lane's V points.
template <int V>
__device__ __forceinline__ void load_spatial(const SpatialArgs& sp, const WaveAddr& w, double (&rate)[V],
                                             double (&srcw)[V]) {
  if (sp.rate) {
    load_v<true, double, V>(at(sp.rate + w.pw, w.ox), V, rate);
  } else {
#pragma unroll
    for (int v = 0; v < V; ++v) rate[v] = 0.0;
  }
  const int64_t p0 = w.pw + (int64_t)(w.ox / 8);
#pragma unroll
  for (int v = 0; v < V; ++v) srcw[v] = (sp.src < 0 || p0 + v == sp.src) ? 1.0 : 0.0;
}

template <typename MT, typename KT>
struct Bdf2Args {
  const KT* ka;         // kappa_a [d*d][stride] (FP64, or FP32 for an FP32-kappa plan)
  const KT* kb;         // kappa_b or null
  const double* Xn;     // X^n      [c][stride]
  const double* Xm;     // X^{n-1}  [c][stride]
  const double* Xmm;    // X^{n-2}  [c][stride] (shifted mode form; null: zero)
  double* Xo;           // X^{n+1}  [c][stride] (may be Xm or Xmm: a block reads its points before it writes them)
  const MT* Yn;         // Y^n      (m * c * stride elements, tiled; Z^n in the shifted form)
  const MT* Ym;         // Y^{n-1}
  MT* Yo;               // Y^{n+1}  (may be Ym: each lane reads a mode before it writes it)
  double* tau;          // [c][stride] or null
  const double* coef;   // [kNumCoef][m]
  double* part;         // block partials or null
  int64_t npoints, main;   // main, wide: blocks of points at V points a lane, and the blocks that
  int wide;                // take them (split_rounds)
  int64_t stride, tile;
  int m;
  Bdf2Scalars s;
  SpatialArgs sp;
};

// Shape of the component-split kernels: blocks of six waves, one per tensor component and 64 V
// points (in 2-D two such groups), so a block covers 64 V kGroups points.
constexpr int kSplitWaves = 6;
template <int D>
struct SplitShape {
  static constexpr int C = Sym<D>::C;
  static constexpr int kGroups = kSplitWaves / C;
  static constexpr int kThreads = 64 * kSplitWaves;
};

// A wave's place in its block.
struct SplitWave { int lane, s, group; };

// The rounds of a component-split launch.  The first `wide` blocks take `main` blocks of points at
// V points a lane (all of them whole) in turn, or, `chunked`, consecutive ones each; the others take
// the points after them at one point a lane, 64 kGroups a round, beside the first ones: what would be a
// nearly empty last round of wide blocks runs along with the full ones, and the ragged end of the field
// needs no launch of its own.  body(width, wave, first point, points left, half): half alternates, so
// that one barrier a round (between the streams and the solves) is enough for LDS that is kept twice.
template <int D, int V, typename F>
__device__ __forceinline__ void split_rounds(int64_t npoints, int64_t main, int wide, int chunked, F&& body) {
  constexpr int C = Sym<D>::C, N1 = 64 * SplitShape<D>::kGroups;
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const SplitWave sw{(int)threadIdx.x % 64, wid % C, wid / C};
  int half = 0;
  if ((int)blockIdx.x < wide) {
    const int64_t step = chunked ? 1 : wide, end = chunked ? main * (blockIdx.x + 1) / wide : main;
    for (int64_t g = chunked ? main * blockIdx.x / wide : blockIdx.x; g < end; g += step, half ^= 1)
      body(std::integral_constant<int, V>{}, sw, g * (N1 * V), npoints - g * (N1 * V), half);
  } else {
    const int64_t step = (int64_t)(gridDim.x - wide) * N1;
    for (int64_t p = main * (N1 * V) + (int64_t)(blockIdx.x - wide) * N1; p < npoints; p += step, half ^= 1)
      body(std::integral_constant<int, 1>{}, sw, p, npoints - p, half);
  }
}

// Modes 0 .. m - 1 of one component in order: load(k, buf) fills a buffer with mode k, use(k,
// buf) consumes it, A modes are in flight.  The steady part of the loop has no branch: each mode
// waits for its own loads only.
template <int A, typename Buf, typename L, typename U>
__device__ __forceinline__ void stream_modes(int m, L&& load, U&& use) {
  Buf buf[A];
#pragma unroll
  for (int j = 0; j < A; ++j)
    if (j < m) load(j, buf[j]);
  int k = 0;
  for (; k + 2 * A <= m; k += A) {
#pragma unroll
    for (int j = 0; j < A; ++j) {
      use(k + j, buf[j]);
      load(k + A + j, buf[j]);
    }
  }
#pragma unroll
  for (int j = 0; j < A; ++j) {
    if (k + j < m) use(k + j, buf[j]);
    if (k + A + j < m) load(k + A + j, buf[j]);
  }
  k += A;
#pragma unroll
  for (int j = 0; j < A; ++j)
    if (k + j < m) use(k + j, buf[j]);
}

// The factors of one mode, consecutive in the plan's packed table: one scalar load, issued a
// mode ahead.
__device__ __forceinline__ void load_pack(const double* coef, int m, int k, double (&c)[kPack]) {
  const double* p = coef + kNumCoefAll * m + (int64_t)k * kPack;
#pragma unroll
  for (int i = 0; i < kPack; ++i) c[i] = load_uniform(p + i);
}

// The mode stream of component s at a wave's 64 groups of V points: G^ (compensated) and P of
// each point go to LDS for the local solve.
// ZF: the shifted mode form Z_k^j = Y_k^j - beta_k X^{j-1}: the history is read back as
// h^_k = 2 Z_k^n - Z_k^{n-1}/2 + beta_k B with B = 2 X^{n-1} - X^{n-2}/2, and the new level is
// stored as Z_k^{n+1} = d_k h^_k + d_k c_k P - beta_k X^n (still independent of X^{n+1}).
template <int D, typename MT, typename KT, int V, bool APART, bool ZF, int A>
__device__ __forceinline__ void bdf2_stream(const Bdf2Args<MT, KT>& a, const LaneAddr<V, APART>& l, int s, double* shP,
                                            double* shG) {
  const WaveAddr& w = l.w;
  const int64_t st = a.stride, T = a.tile;
  const int m = a.m;
  // P = 2 X^n - X^{n-1}/2 (and B = 2 X^{n-1} - X^{n-2}/2 in the shifted form)
  double xn[V], xm[V], P[V], B[V], Gs[V], Ge[V];
  load_points(a.Xn + s * st + w.pw, l, xn);
  load_points(a.Xm + s * st + w.pw, l, xm);
  if constexpr (ZF) {
    double xmm[V];
    if (a.Xmm) {
      load_points(a.Xmm + s * st + w.pw, l, xmm);
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) xmm[v] = 0.0;
    }
#pragma unroll
    for (int v = 0; v < V; ++v) B[v] = 2.0 * xm[v] - 0.5 * xmm[v];
  }
#pragma unroll
  for (int v = 0; v < V; ++v) {
    P[v] = 2.0 * xn[v] - 0.5 * xm[v];
    Gs[v] = 0.0;
    Ge[v] = 0.0;
  }
  const MT* yn0 = a.Yn + w.tw + s * T;
  const MT* ym0 = a.Ym + w.tw + s * T;
  MT* yo0 = a.Yo + w.tw + s * T;
  const int64_t kT = (int64_t)Sym<D>::C * T;
  double pack[kPack];
  load_pack(a.coef, m, 0, pack);
  struct Buf { MT n[V], m[V]; };
  stream_modes<A, Buf>(
      m,
      [&](int k, Buf& b) {
        load_modes(yn0 + k * kT, l, b.n);
        load_modes(ym0 + k * kT, l, b.m);
      },
      [&](int k, const Buf& b) {
        const double dk = pack[kPackD], dck = pack[kPackDC], ek = pack[kPackEta], bk = pack[kPackBeta];
        load_pack(a.coef, m, k + 1 < m ? k + 1 : k, pack);
        MT out[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
          double h = 2.0 * (double)b.n[v] - 0.5 * (double)b.m[v];
          if constexpr (ZF) {
            h += bk * B[v];
            out[v] = (MT)(dk * h + (dck * P[v] - bk * xn[v]));
          } else {
            out[v] = (MT)(dk * h + dck * P[v]);
          }
          two_sum_acc(Gs[v], Ge[v], mul_rn(ek, h));
        }
        store_modes(yo0 + k * kT, l, out);
      });
#pragma unroll
  for (int v = 0; v < V; ++v) {
    shP[v * l.kStep] = P[v];
    shG[v * l.kStep] = Gs[v] + Ge[v];
  }
}

// The velocity gradient driving the step at one point, in its storage precision.
template <int D, typename KT>
struct KappaAt {
  KT a[D * D], b[D * D];
  template <typename Args>
  __device__ __forceinline__ void load(const Args& A, int64_t pw, uint32_t q) {
    const uint32_t kx = q * (uint32_t)sizeof(KT);
#pragma unroll
    for (int t = 0; t < D * D; ++t) a[t] = *at(A.ka + t * A.stride + pw, kx);
    if (A.kb) {
#pragma unroll
      for (int t = 0; t < D * D; ++t) b[t] = *at(A.kb + t * A.stride + pw, kx);
    }
  }
};

// The local solve of one point: kappa~, R, X^{n+1} and tau (SPLIT: R and G, no solve), from its
// P and G^ in LDS.
template <int D, typename MT, typename KT, int NP, bool DIAG, bool SP, bool SPLIT>
__device__ __forceinline__ void bdf2_point(const Bdf2Args<MT, KT>& a, int64_t pw, uint32_t q,
                                           const KappaAt<D, KT>& kap, const double* shP, const double* shG,
                                           DiagAcc& acc) {
  constexpr int C = Sym<D>::C;
  const int64_t st = a.stride;
  const uint32_t ox = q * 8;
  // velocity gradient driving the step (read in its storage precision, extrapolated in FP64)
  double k[D * D], P[C], G[C], AG[C], R[C];
#pragma unroll
  for (int t = 0; t < D * D; ++t) k[t] = a.kb ? 2.0 * (double)kap.a[t] - (double)kap.b[t] : (double)kap.a[t];
  double rate = 0.0, srcw = 1.0;
  if constexpr (SP) {
    if (a.sp.rate) rate = *at(a.sp.rate + pw, ox);
    srcw = (a.sp.src < 0 || pw + (int64_t)q == a.sp.src) ? 1.0 : 0.0;
  }
  // relaxation plus the spatial rate; the mass-mode source; the diagonal of M
  const double idv = SP ? a.s.inv_De + rate : a.s.inv_De;
  const double zw = SP ? a.s.zeta * srcw : a.s.zeta;
  const double ad = SP ? a.s.a_diag + a.s.eta * rate : a.s.a_diag;
#pragma unroll
  for (int s = 0; s < C; ++s) {
    P[s] = shP[s * NP];
    G[s] = shG[s * NP] + a.s.s_ec * P[s];
  }
  apply_K<D>(k, G, AG);
#pragma unroll
  for (int s = 0; s < C; ++s) {
    const int i = Sym<D>::i(s), j = Sym<D>::j(s);
    const double S = k[i * D + j] + k[j * D + i];
    R[s] = P[s] - (AG[s] - idv * G[s]) + zw * S;
  }
  double ts[C];
  if constexpr (SPLIT) {
#pragma unroll
    for (int s = 0; s < C; ++s) ts[s] = G[s];
  } else {
    double M[C][C];
    build_M<D>(k, ad, a.s.eta, M);
    solve_pivot<C>(M, R);
#pragma unroll
    for (int s = 0; s < C; ++s) ts[s] = a.s.tau_scale * (a.s.eta * R[s] - G[s]);
    if constexpr (DIAG) diag_point<D>(acc, R, ts);
  }
#pragma unroll
  for (int s = 0; s < C; ++s) {
    *at(a.Xo + s * st + pw, ox) = R[s];
    if (a.tau) *at(a.tau + s * st + pw, ox) = ts[s];
  }
}

// The step in blocks of six waves, one per tensor component: the mode stream of a component needs
// no other one, so a wave holds one component's sums and a few modes ahead, and a small grid has
// c times the waves.  Then one lane per point solves the c x c system; the LDS of consecutive
// rounds alternates, so one barrier a round is enough.  Every point's arithmetic and its order
// are the same for every V.
// Bound: HBM on whole grids (3-D, m = 32, FP32 modes, 128^3: 884 us, 0.76 of 8 TB/s; a lane that
// held all six components of its points: 906 us at one or two waves per SIMD), latency on small
// ones (4096 points, 2-D, m = 32, FP64: 8.6 us, was 18.6; 45^3 points, 3-D, m = 40, FP32: 53 us,
// was 113 with its own launch for the last point).  A few modes ahead are enough: twice as many
// cost 3% at 128^3, and so do the next points' loads during the solve.
// SPLIT: the step without its local solve, for a caller that solves a spatially coupled
// system for X^{n+1}: the modes advance as usual (in the Y-form they do not depend on
// X^{n+1}), the point's right-hand side R goes to Xo and the history combination G to tau.
template <int D, typename MT, typename KT, int V, bool APART, bool DIAG, bool SP, bool SPLIT = false, bool ZF = false>
__global__ __launch_bounds__(SplitShape<D>::kThreads) void bdf2_kernel(const Bdf2Args<MT, KT> a) {
  constexpr int C = Sym<D>::C;
  __shared__ double sh[2][2 * C * SplitShape<D>::kGroups * 64 * V];
  DiagAcc acc;
  split_rounds<D, V>(a.npoints, a.main, a.wide, 0, [&](auto width, const SplitWave& sw, int64_t pw, int64_t left, int half) {
    constexpr int W = decltype(width)::value, NP = SplitShape<D>::kGroups * 64 * W, T = SplitShape<D>::kThreads;
    constexpr int Q = (NP + T - 1) / T, A = sizeof(MT) * W >= 16 ? 2 : 4;
    KappaAt<D, KT> kap[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int q = threadIdx.x + i * T;
      if (q < NP && q < left) kap[i].load(a, pw, q);
    }
    double* shP = sh[half];
    double* shG = shP + C * NP;
    using L = LaneAddr<W, APART && W != 1>;
    const int p1 = sw.group * 64 * W, o = sw.s * NP + p1 + sw.lane * L::kLane;
    if (p1 + sw.lane * L::kLane < left)
      bdf2_stream<D, MT, KT, W, APART && W != 1, ZF, A>(
          a, lane_addr<MT, C, W, APART && W != 1>(pw + p1, sw.lane, a.tile, a.m), sw.s, shP + o, shG + o);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int q = threadIdx.x + i * T;
      if (q < NP && q < left) bdf2_point<D, MT, KT, NP, DIAG, SP, SPLIT>(a, pw, q, kap[i], shP + q, shG + q, acc);
    }
  });
  if constexpr (DIAG) {
    const DiagAcc r = block_reduce<kSplitWaves>(acc);
    if (threadIdx.x == 0) write_partial(a.part, blockIdx.x, r);
  }
}

// The 2-D FP64 step with one lane per two points and all three components, for whole grids: there
// three components and two points fit a lane's registers at two waves per SIMD, each wave's
// accesses are consecutive planes, and the step streams 4% faster than in component waves (1024^2,
// m = 32: 397 us, 0.81 of 8 TB/s, against 413).  npoints is even.
template <bool DIAG, bool SP, bool SPLIT>
__device__ __forceinline__ void bdf2_wide_group(const Bdf2Args<double, double>& a, const WaveAddr& w, DiagAcc& acc) {
  constexpr int D = 2, C = 3, V = 2;
  const int64_t st = a.stride;
  const int m = a.m;
  const int64_t T = a.tile;

  // P = 2 X^n - X^{n-1}/2
  double P[C][V];
#pragma unroll
  for (int s = 0; s < C; ++s) {
    double xn[V], xm[V];
    load_v<true, double, V>(at(a.Xn + s * st + w.pw, w.ox), V, xn);
    load_v<true, double, V>(at(a.Xm + s * st + w.pw, w.ox), V, xm);
#pragma unroll
    for (int v = 0; v < V; ++v) P[s][v] = 2.0 * xn[v] - 0.5 * xm[v];
  }

  // mode stream: the loads of mode k+1 are issued before the stores of mode k
  double Gs[C][V], Ge[C][V];
#pragma unroll
  for (int s = 0; s < C; ++s)
#pragma unroll
    for (int v = 0; v < V; ++v) { Gs[s][v] = 0.0; Ge[s][v] = 0.0; }

  const double* yn0 = a.Yn + w.tw;
  const double* ym0 = a.Ym + w.tw;
  double* yo0 = a.Yo + w.tw;
  double cn[C][V], cm[C][V];
#pragma unroll
  for (int s = 0; s < C; ++s) {
    load_v<true, double, V, true>(at(yn0 + s * T, w.om), V, cn[s]);
    load_v<true, double, V, true>(at(ym0 + s * T, w.om), V, cm[s]);
  }
  for (int k = 0; k < m; ++k) {
    const double dk = load_uniform(a.coef + kRowD * m + k);
    const double dck = load_uniform(a.coef + kRowDC * m + k);
    const double ek = load_uniform(a.coef + kRowEta * m + k);
    double nn[C][V], nm[C][V];
    if (k + 1 < m) {
      const int64_t o = (int64_t)(k + 1) * C * T;
      const uint32_t om = opaque(w.om);
#pragma unroll
      for (int s = 0; s < C; ++s) {
        load_v<true, double, V, true>(at(yn0 + o + s * T, om), V, nn[s]);
        load_v<true, double, V, true>(at(ym0 + o + s * T, om), V, nm[s]);
      }
    }
    double* yo = yo0 + (int64_t)k * C * T;
    const uint32_t om = opaque(w.om);
#pragma unroll
    for (int s = 0; s < C; ++s) {
      double out[V];
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const double h = 2.0 * cn[s][v] - 0.5 * cm[s][v];
        out[v] = dk * h + dck * P[s][v];
        two_sum_acc(Gs[s][v], Ge[s][v], mul_rn(ek, h));
      }
      store_v<true, double, V, true>(at(yo + s * T, om), V, out);
    }
    if (k + 1 < m) {
#pragma unroll
      for (int s = 0; s < C; ++s)
#pragma unroll
        for (int v = 0; v < V; ++v) { cn[s][v] = nn[s][v]; cm[s][v] = nm[s][v]; }
    }
  }

  // velocity gradient driving the step
  double kt[D * D][V];
#pragma unroll
  for (int q = 0; q < D * D; ++q) {
    double ka[V];
    load_v<true, double, V>(at(a.ka + q * st + w.pw, w.ox), V, ka);
    if (a.kb) {
      double kb[V];
      load_v<true, double, V>(at(a.kb + q * st + w.pw, w.ox), V, kb);
#pragma unroll
      for (int v = 0; v < V; ++v) kt[q][v] = 2.0 * ka[v] - kb[v];
    } else {
#pragma unroll
      for (int v = 0; v < V; ++v) kt[q][v] = ka[v];
    }
  }

  double rate[V], srcw[V];
  if constexpr (SP) load_spatial<V>(a.sp, w, rate, srcw);
  double Xout[C][V], Tout[C][V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    double k[D * D], G[C], AG[C], R[C];
    // relaxation plus the spatial rate; the mass-mode source; the diagonal of M
    const double idv = SP ? a.s.inv_De + rate[v] : a.s.inv_De;
    const double zw = SP ? a.s.zeta * srcw[v] : a.s.zeta;
    const double ad = SP ? a.s.a_diag + a.s.eta * rate[v] : a.s.a_diag;
#pragma unroll
    for (int q = 0; q < D * D; ++q) k[q] = kt[q][v];
#pragma unroll
    for (int s = 0; s < C; ++s) G[s] = (Gs[s][v] + Ge[s][v]) + a.s.s_ec * P[s][v];
    apply_K<D>(k, G, AG);
#pragma unroll
    for (int s = 0; s < C; ++s) {
      const int i = Sym<D>::i(s), j = Sym<D>::j(s);
      const double S = k[i * D + j] + k[j * D + i];
      R[s] = P[s][v] - (AG[s] - idv * G[s]) + zw * S;
    }
    if constexpr (SPLIT) {
#pragma unroll
      for (int s = 0; s < C; ++s) {
        Xout[s][v] = R[s];
        Tout[s][v] = G[s];
      }
      continue;
    }
    double M[C][C];
    build_M<D>(k, ad, a.s.eta, M);
    solve_pivot<C>(M, R);
#pragma unroll
    for (int s = 0; s < C; ++s) {
      Xout[s][v] = R[s];
      Tout[s][v] = a.s.tau_scale * (a.s.eta * R[s] - G[s]);
    }
    if constexpr (DIAG) {
      double xs[C], ts[C];
#pragma unroll
      for (int s = 0; s < C; ++s) { xs[s] = Xout[s][v]; ts[s] = Tout[s][v]; }
      diag_point<D>(acc, xs, ts);
    }
  }
#pragma unroll
  for (int s = 0; s < C; ++s) {
    store_v<true, double, V>(at(a.Xo + s * st + w.pw, w.ox), V, Xout[s]);
    if (a.tau) store_v<true, double, V>(at(a.tau + s * st + w.pw, w.ox), V, Tout[s]);
  }
}

template <bool DIAG, bool SP, bool SPLIT>
__global__ __launch_bounds__(kBlock) void bdf2_wide_kernel(const Bdf2Args<double, double> a) {
  DiagAcc acc;
  const int lane = threadIdx.x % 64;
  const int64_t ngroups = a.npoints / 2, nwaves = (ngroups + 63) / 64;
  const int64_t wstride = (int64_t)gridDim.x * (kBlock / 64);
  for (int64_t wv = wave_uniform((int64_t)blockIdx.x * (kBlock / 64) + threadIdx.x / 64); wv < nwaves;
       wv += wstride) {
    if (wv * 64 + lane < ngroups)
      bdf2_wide_group<DIAG, SP, SPLIT>(a, wave_addr<double, 3, 2>(wv * 128, lane, a.tile, a.m), acc);
  }
  if constexpr (DIAG) {
    const DiagAcc r = block_reduce<kBlock / 64>(acc);
    if (threadIdx.x == 0) write_partial(a.part, blockIdx.x, r);
  }
}

// ------------------------------------------------------------------ SDIRK2 start-up
template <typename MT, typename KT>
struct StartArgs {
  const KT* ka;      // kappa^0
  const double* X0;  // X^0 [c][stride]
  double* X1;        // X^1 [c][stride] (out)
  MT* Y0;            // Y^0 (m * c * stride elements, tiled; out)
  MT* Y1;            // Y^1 (out)
  double* tau;
  const double* coef;
  double* part;
  int64_t p_begin, ngroups;
  int64_t stride, tile;
  int m, part0;
  int zform;         // shifted mode form: Z^1 = Y^1 - beta_k X^0 (Z^0 = Y^0: X^{-1} = 0)
  StartScalars s;
  SpatialArgs sp;
};

template <int D, typename MT, typename KT, int V, bool DIAG, bool SP>
__device__ __forceinline__ void start_group(const StartArgs<MT, KT>& a, const WaveAddr& w, DiagAcc& acc) {
  constexpr int C = Sym<D>::C;
  const int64_t st = a.stride;
  const int m = a.m;
  double X0[C][V], X1[C][V], X2[C][V];
#pragma unroll
  for (int s = 0; s < C; ++s) load_v<true, double, V>(at(a.X0 + s * st + w.pw, w.ox), V, X0[s]);
  double kt[D * D][V];
#pragma unroll
  for (int q = 0; q < D * D; ++q) {
    KT x[V];
    load_v<true, KT, V>(at(a.ka + q * st + w.pw, field_off<KT>(w.ox)), V, x);
#pragma unroll
    for (int v = 0; v < V; ++v) kt[q][v] = (double)x[v];
  }

  double rate[V], srcw[V];
  if constexpr (SP) load_spatial<V>(a.sp, w, rate, srcw);
  double Tout[C][V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    double k[D * D], S[C], r[C], M[C][C], AX[C], x1[C];
    // relaxation plus the spatial rate; the mass-mode source of the two stages
    const double idv = SP ? a.s.inv_De + rate[v] : a.s.inv_De;
    const double s1 = SP ? a.s.src1 * srcw[v] : a.s.src1;
    const double s2 = SP ? a.s.sigma2 * srcw[v] : a.s.sigma2;
#pragma unroll
    for (int q = 0; q < D * D; ++q) k[q] = kt[q][v];
#pragma unroll
    for (int s = 0; s < C; ++s) {
      const int i = Sym<D>::i(s), j = Sym<D>::j(s);
      S[s] = k[i * D + j] + k[j * D + i];
    }
    // stage 1: (I - h gs theta A) X1 = X0 + h gs theta S
#pragma unroll
    for (int s = 0; s < C; ++s) r[s] = X0[s][v] + s1 * S[s];
    build_M<D>(k, 1.0 + a.s.hgt * idv, a.s.hgt, M);
    solve_pivot<C>(M, r);
#pragma unroll
    for (int s = 0; s < C; ++s) { x1[s] = r[s]; X1[s][v] = r[s]; }
    // stage 2: (I - h gs theta A) X2 = X0 + sigma1 A(X1) + sigma2 S
    apply_K<D>(k, x1, AX);
#pragma unroll
    for (int s = 0; s < C; ++s)
      r[s] = X0[s][v] + a.s.sigma1 * (AX[s] - idv * x1[s]) + s2 * S[s];
    build_M<D>(k, 1.0 + a.s.hgt * idv, a.s.hgt, M);
    solve_pivot<C>(M, r);
#pragma unroll
    for (int s = 0; s < C; ++s) {
      X2[s][v] = r[s];
      Tout[s][v] = a.s.gamma * (a.s.theta * r[s] - a.s.hr * x1[s]);
    }
    if constexpr (DIAG) {
      double xs[C], ts[C];
#pragma unroll
      for (int s = 0; s < C; ++s) { xs[s] = X2[s][v]; ts[s] = Tout[s][v]; }
      diag_point<D>(acc, xs, ts);
    }
  }
#pragma unroll
  for (int s = 0; s < C; ++s) {
    store_v<true, double, V>(at(a.X1 + s * st + w.pw, w.ox), V, X2[s]);
    if (a.tau) store_v<true, double, V>(at(a.tau + s * st + w.pw, w.ox), V, Tout[s]);
  }
  // modes: Y_k^0 = -c_k X^0 (slot 0), Y_k^1 = u_k X^(1) + v_k X^(2) (slot 1); in the
  // shifted form level 1 is stored less beta_k X^0
  const int64_t T = a.tile;
  MT* Y0 = a.Y0 + w.tw;
  MT* Y1 = a.Y1 + w.tw;
  for (int k = 0; k < m; ++k) {
    const double ck = load_uniform(a.coef + kRowC * m + k);
    const double uk = load_uniform(a.coef + kRowU * m + k);
    const double vk = load_uniform(a.coef + kRowV * m + k);
    const double bk = a.zform ? load_uniform(a.coef + kRowBeta * m + k) : 0.0;
#pragma unroll
    for (int s = 0; s < C; ++s) {
      MT o0[V], o1[V];
#pragma unroll
      for (int v = 0; v < V; ++v) {
        o0[v] = (MT)(-ck * X0[s][v]);
        o1[v] = (MT)((uk * X1[s][v] + vk * X2[s][v]) - bk * X0[s][v]);
      }
      store_v<true, MT, V, true>(at(Y0 + ((int64_t)k * C + s) * T, w.om), V, o0);
      store_v<true, MT, V, true>(at(Y1 + ((int64_t)k * C + s) * T, w.om), V, o1);
    }
  }
}

template <int D, typename MT, typename KT, int V, bool DIAG, bool SP>
__global__ __launch_bounds__(kBlock) void start_kernel(const StartArgs<MT, KT> a) {
  constexpr int C = Sym<D>::C;
  DiagAcc acc;
  const int lane = threadIdx.x % 64;
  const int64_t nwaves = (a.ngroups + 63) / 64;
  const int64_t wstride = (int64_t)gridDim.x * (kBlock / 64);
  for (int64_t wv = wave_uniform((int64_t)blockIdx.x * (kBlock / 64) + threadIdx.x / 64); wv < nwaves;
       wv += wstride) {
    if (wv * 64 + lane < a.ngroups)
      start_group<D, MT, KT, V, DIAG, SP>(a, wave_addr<MT, C, V>(a.p_begin + wv * 64 * V, lane, a.tile, a.m), acc);
  }
  if constexpr (DIAG) {
    const DiagAcc r = block_reduce<kBlock / 64>(acc);
    if (threadIdx.x == 0) write_partial(a.part, a.part0 + blockIdx.x, r);
  }
}

// ------------------------------------------------------------------ exponential-mode step
// Each mode is advanced exactly for X linear on the step (TFS_SCHEME_EXP):
//   Y_k^{n+1} = e_k Y_k^n + f_k X^n                      (Y_k = X_k - q_k X, stored in place)
//   H  = sum_k (1 - e_k) Y_k^n + s_h X^n                  (X^{n+1} - X^n = A(q X^{n+1} - H) + zeta S)
//   G  = sum_k lambda_k dt Y_k^{n+1}                      (dt D^{1-alpha} X^{n+1} = eta_e X^{n+1} - G)
//   [(1 + q/De) I - q (kappa~ . + . kappa~^T)] X^{n+1} = X^n - A(H) + zeta S
//   tau^{n+1} = (gamma/dt)(eta_e X^{n+1} - G)
// H and G are compensated FP64 sums; one read and one write per mode-component.

template <typename MT, typename KT>
struct ExpArgs {
  const KT* ka;         // kappa_a [d*d][stride]
  const KT* kb;         // kappa_b or null
  const double* Xn;     // X^n     [c][stride]
  double* Xo;           // X^{n+1} [c][stride]
  const MT* Yn;         // Y^n (m * c * stride elements, tiled); not read at n = 0
  MT* Yo;               // Y^{n+1} (may be Yn: each lane reads a mode before writing it)
  double* tau;          // [c][stride] or null
  double* Hout;         // SPLIT: H [c][stride]
  const double* coef;   // [kNumCoef][m], ExpRow order
  double* part;         // block partials or null
  int64_t npoints, main;   // main, wide: blocks of points at V points a lane, and the blocks that
  int wide;                // take them, consecutive ones a block where chunked (split_rounds)
  int chunked;
  int64_t stride, tile;
  int m;
  ExpScalars s;
  SpatialArgs sp;
};

// The mode stream of component s at a wave's 64 groups of V points; H enters the solve only
// (plain FP64 sum), G is the stress's near-cancelling term (compensated).
template <int D, typename MT, typename KT, int V, bool APART, int A>
__device__ __forceinline__ void exp_stream(const ExpArgs<MT, KT>& a, const LaneAddr<V, APART>& l, int s, double* shX,
                                           double* shH, double* shG) {
  const WaveAddr& w = l.w;
  const int64_t T = a.tile;
  const int m = a.m;
  const bool first = a.s.first != 0;
  double Xc[V], H[V], Gs[V], Ge[V];
  load_points(a.Xn + s * a.stride + w.pw, l, Xc);
#pragma unroll
  for (int v = 0; v < V; ++v) { H[v] = 0.0; Gs[v] = 0.0; Ge[v] = 0.0; }
  const MT* yn0 = a.Yn + w.tw + s * T;
  MT* yo0 = a.Yo + w.tw + s * T;
  const int64_t kT = (int64_t)Sym<D>::C * T;
  double pack[kPack];
  load_pack(a.coef, m, 0, pack);
  struct Buf { MT y[V]; };
  auto use = [&](int k, const Buf& b) {
    const double ek = pack[kPackE], fk = pack[kPackF], lk = pack[kPackLdt], ok = pack[kPackOneME], qk = pack[kPackQ];
    load_pack(a.coef, m, k + 1 < m ? k + 1 : k, pack);
    MT out[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const double y = first ? -qk * Xc[v] : (double)b.y[v];
      out[v] = (MT)(ek * y + fk * Xc[v]);
      H[v] += ok * y;
      two_sum_acc(Gs[v], Ge[v], mul_rn(lk, (double)out[v]));
    }
    store_modes(yo0 + k * kT, l, out);
  };
  if (first) {   // level 0's modes are -q_k X^0: nothing to read
    for (int k = 0; k < m; ++k) use(k, Buf{});
  } else {
    stream_modes<A, Buf>(m, [&](int k, Buf& b) { load_modes(yn0 + k * kT, l, b.y); }, use);
  }
#pragma unroll
  for (int v = 0; v < V; ++v) {
    shX[v * l.kStep] = Xc[v];
    shH[v * l.kStep] = H[v];
    shG[v * l.kStep] = Gs[v] + Ge[v];
  }
}

// The local solve of one point (SPLIT: R, G and H, no solve), from X^n, H and G in LDS.
template <int D, typename MT, typename KT, int NP, bool DIAG, bool SP, bool SPLIT>
__device__ __forceinline__ void exp_point(const ExpArgs<MT, KT>& a, int64_t pw, uint32_t q,
                                          const KappaAt<D, KT>& kap, const double* shX, const double* shH,
                                          const double* shG, DiagAcc& acc) {
  constexpr int C = Sym<D>::C;
  const int64_t st = a.stride;
  const uint32_t ox = q * 8;
  double k[D * D], Xc[C], Hv[C], AH[C], R[C], ts[C];
#pragma unroll
  for (int t = 0; t < D * D; ++t)
    k[t] = a.kb ? a.s.fa * (double)kap.a[t] + a.s.fb * (double)kap.b[t] : (double)kap.a[t];
  double rate = 0.0, srcw = 1.0;                 // spatial form: extra rate, source weight
  if constexpr (SP) {
    if (a.sp.rate) rate = *at(a.sp.rate + pw, ox);
    srcw = (a.sp.src < 0 || pw + (int64_t)q == a.sp.src) ? 1.0 : 0.0;
  }
  const double idv = SP ? a.s.inv_De + rate : a.s.inv_De;
  const double zw = SP ? a.s.zeta * srcw : a.s.zeta;
  const double ad = SP ? a.s.a_diag + a.s.q * rate : a.s.a_diag;
#pragma unroll
  for (int s = 0; s < C; ++s) {
    Xc[s] = shX[s * NP];
    Hv[s] = shH[s * NP] + a.s.s_h * Xc[s];
  }
  apply_K<D>(k, Hv, AH);
#pragma unroll
  for (int s = 0; s < C; ++s) {
    const int i = Sym<D>::i(s), j = Sym<D>::j(s);
    const double S = k[i * D + j] + k[j * D + i];
    R[s] = Xc[s] - (AH[s] - idv * Hv[s]) + zw * S;
  }
  if constexpr (SPLIT) {
#pragma unroll
    for (int s = 0; s < C; ++s) {
      ts[s] = shG[s * NP];
      *at(a.Hout + s * st + pw, ox) = Hv[s];
    }
  } else {
    double M[C][C];
    build_M<D>(k, ad, a.s.q, M);
    solve_pivot<C>(M, R);
#pragma unroll
    for (int s = 0; s < C; ++s) ts[s] = a.s.tau_scale * (a.s.eta_e * R[s] - shG[s * NP]);
    if constexpr (DIAG) diag_point<D>(acc, R, ts);
  }
#pragma unroll
  for (int s = 0; s < C; ++s) {
    *at(a.Xo + s * st + pw, ox) = R[s];
    if (a.tau) *at(a.tau + s * st + pw, ox) = ts[s];
  }
}

// Blocks, waves and lanes as in bdf2_kernel (3-D, m = 32, FP32 modes, 128^3: 654 us, 0.73 of
// 8 TB/s, was 660; 4096 points, 2-D, FP64: 8.7 us, was 18.3).  The first step only writes modes
// (884736 points, FP32 modes: 149 us, bound by its stores).
// SPLIT: the step without its local solve, for a caller that solves a spatially coupled
// system: X^{n+1} receives each point's right-hand side R, tau the compensated G and Hout the
// H of the local system (the modes are written as usual: they do not depend on X^{n+1}).
template <int D, typename MT, typename KT, int V, bool APART, bool DIAG, bool SP, bool SPLIT = false>
__global__ __launch_bounds__(SplitShape<D>::kThreads) void exp_kernel(const ExpArgs<MT, KT> a) {
  constexpr int C = Sym<D>::C;
  __shared__ double sh[2][3 * C * SplitShape<D>::kGroups * 64 * V];
  DiagAcc acc;
  split_rounds<D, V>(a.npoints, a.main, a.wide, a.chunked, [&](auto width, const SplitWave& sw, int64_t pw, int64_t left, int half) {
    constexpr int W = decltype(width)::value, NP = SplitShape<D>::kGroups * 64 * W, T = SplitShape<D>::kThreads;
    constexpr int Q = (NP + T - 1) / T, A = sizeof(MT) * W >= 16 ? 4 : 8;
    KappaAt<D, KT> kap[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int q = threadIdx.x + i * T;
      if (q < NP && q < left) kap[i].load(a, pw, q);
    }
    double* shX = sh[half];
    double* shH = shX + C * NP;
    double* shG = shH + C * NP;
    using L = LaneAddr<W, APART && W != 1>;
    const int p1 = sw.group * 64 * W, o = sw.s * NP + p1 + sw.lane * L::kLane;
    if (p1 + sw.lane * L::kLane < left)
      exp_stream<D, MT, KT, W, APART && W != 1, A>(
          a, lane_addr<MT, C, W, APART && W != 1>(pw + p1, sw.lane, a.tile, a.m), sw.s, shX + o, shH + o, shG + o);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < Q; ++i) {
      const int q = threadIdx.x + i * T;
      if (q < NP && q < left)
        exp_point<D, MT, KT, NP, DIAG, SP, SPLIT>(a, pw, q, kap[i], shX + q, shH + q, shG + q, acc);
    }
  });
  if constexpr (DIAG) {
    const DiagAcc r = block_reduce<kSplitWaves>(acc);
    if (threadIdx.x == 0) write_partial(a.part, blockIdx.x, r);
  }
}

// ------------------------------------------------------------------ plain modes
// X_k = Y_k + c_k X^j (+ beta_k X^{j-1} in the shifted form, Xm null: zero).
template <typename MT>
__global__ __launch_bounds__(kBlock) void plain_kernel(const double* __restrict__ X, const double* __restrict__ Xm,
                                                       const MT* __restrict__ Y, const double* __restrict__ coef,
                                                       double* __restrict__ out, int64_t npts, int64_t stride,
                                                       int64_t tile, int m, int c, int zform) {
  const int64_t total = (int64_t)m * c * npts;
  for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < total; t += (int64_t)gridDim.x * kBlock) {
    const int64_t p = t % npts;
    const int64_t ks = t / npts;
    const int s = (int)(ks % c);
    const int k = (int)(ks / c);
    const int64_t yi = ((p / tile) * m * c + ks) * tile + p % tile;
    double x = (double)Y[yi] + coef[kRowC * m + k] * X[s * stride + p];
    if (zform && Xm) x += coef[kRowBeta * m + k] * Xm[s * stride + p];
    out[ks * stride + p] = x;
  }
}

// ------------------------------------------------------------------ launch helpers
int grid_for(const tfs_plan_s* p, int64_t ngroups) {
  const int64_t cap = (int64_t)p->num_cus * p->grid_per_cu;
  int64_t g = (ngroups + kBlock - 1) / kBlock;
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  return (int)g;
}

bool aligned(const void* ptr, size_t bytes) { return ptr == nullptr || ((uintptr_t)ptr % bytes) == 0; }

// Points per lane and access: the requested width, else the widest up to `widest` for which every plane start
// and every group start is aligned to the vector size of each field (modes: V * sizeof(MT); the
// other fields, FP64: V * 8).  widest: a lane loads 16 bytes of a mode or more (FP64: 2 points;
// FP32: 2 points of BDF2's two levels, 4 of the exponential scheme's one); wider lanes only hold
// more registers (884736 points in 3-D, m = 48, FP32, BDF2: 531 us with 2, 539 with 4; 128^3
// exponential, m = 32: 742 with 2, 683 with 4).
template <int D, typename MT, typename KT>
int pick_vec(const tfs_plan_s* p, const void* k0, const void* k1, const Levels& L, const void* tau, int widest) {
  for (int V = sizeof(MT) == 4 ? 4 : 2; V > 1; V /= 2) {
    if (p->vec_override ? V != p->vec_override : V > widest) continue;
    if (p->stride % V || p->tile % V) continue;
    const size_t bm = (size_t)V * sizeof(MT), bd = (size_t)V * 8, bk = (size_t)V * sizeof(KT);
    if (aligned(k0, bk) && aligned(k1, bk) && aligned(L.Xn, bd) && aligned(L.Xm, bd) && aligned(L.Xmm, bd) &&
        aligned(L.Xo, bd) && aligned(L.Yn, bm) && aligned(L.Ym, bm) && aligned(L.Ym0, bm) && aligned(L.Yo, bm) &&
        aligned(tau, bd) && aligned(p->sp_rate, bd))
      return V;
  }
  return 1;
}

// The grid of a component-split launch (split_rounds): its blocks, the wide ones among them, and
// the wide blocks of points.  At most step_grid blocks per CU of either kind: one by default, whose
// six waves keep enough loads in flight; more resident blocks only add streams (884736 points,
// 3-D, m = 48, FP32: 531 us with one, 546 with eleven).  A last round of wide blocks over fewer
// than three quarters of the CUs goes to the narrow ones.
struct SplitGrid { int grid, wide; int64_t main; };

SplitGrid split_grid(const tfs_plan_s* p, int V) {
  const int64_t n1 = 64 * (kSplitWaves / p->c), cap = (int64_t)p->num_cus * p->step_grid;
  const int64_t whole = p->npoints / (n1 * V), extra = whole % cap;
  const int64_t main = 4 * extra >= 3 * cap ? whole : whole - extra;
  const int64_t narrow = (p->npoints - main * n1 * V + n1 - 1) / n1;
  const int64_t wide = std::min(cap, main);
  return {(int)(wide + std::min(cap, narrow)), (int)wide, main};
}

// Whether an exponential step's blocks take consecutive blocks of points: large 3-D FP64 grids (m = 40,
// 2^24 points 11883 us in turn, 10903 so; 2^22 2898 and 2860; but 884736 points, m = 32, 451 and 467).
template <int D, typename MT>
int chunked_rounds(const tfs_plan_s* p) { return D == 3 && sizeof(MT) == 8 && p->npoints >= (1 << 21); }

// The mean share of the CUs that is busy when blocks of `per` points go round by round.
double fill(const tfs_plan_s* p, int64_t per) {
  const double rounds = (double)((p->npoints + per - 1) / per) / p->num_cus;
  return rounds / std::ceil(rounds);
}

// Where the alignment allows no wide access a step of whole blocks still takes several points a lane,
// each with its own access (LaneAddr, APART): a wave visits 1 KB of a mode plane at a time.  With one
// point a lane it visits 256 bytes, which start and end within cache lines that other blocks share
// (odd stride, m = 32, 262145 points, 3-D: FP32 exponential 152 us against 100, FP32 BDF2 199 against
// 140, FP64 BDF2 286 against 260).  A grid of narrow rounds only keeps the smaller kernel (20001 points,
// 3-D, FP32 BDF2: 19 us against 24).
template <typename MT>
constexpr int kApart = sizeof(MT) == 4 ? 4 : 2;

template <typename MT>
bool points_apart(const tfs_plan_s* p) {
  return p->vec_override != 1 && split_grid(p, kApart<MT>).main > 0;
}

// Whether a step takes bdf2_wide_kernel: 2-D FP64 plans without a shifted form, two points a lane,
// and enough points for two rounds of its blocks of 512 with the last round nearly full (262144
// points, m = 32: 103 us against 108; 200001: 110 against 87, one round and a half).
template <int D, typename MT, typename KT>
bool wide_step(const tfs_plan_s* p, int V) {
  if constexpr (D == 2 && sizeof(MT) == 8)
    return V == 2 && !p->zform && p->npoints % 2 == 0 && p->npoints >= (int64_t)2 * 512 * p->num_cus &&
           fill(p, 512) >= 0.95;
  return false;
}

int wide_blocks(const tfs_plan_s* p) {
  const int64_t cap = (int64_t)p->num_cus * p->step_grid, g = (p->npoints + 511) / 512;
  return (int)(g < cap ? g : cap);
}

template <int D, typename MT, typename KT, int V, bool APART, bool DIAG, bool SP, bool ZF>
hipError_t bdf2_go_(const tfs_plan_s* p, Bdf2Args<MT, KT> a, double* diag_out) {
  const SplitGrid sg = split_grid(p, V);
  int grid = sg.grid;
  a.main = sg.main;
  a.wide = sg.wide;
  bool wide = false;
  if constexpr (D == 2 && sizeof(MT) == 8 && !ZF && !APART) {
    if ((wide = wide_step<D, MT, KT>(p, V))) {
      grid = wide_blocks(p);
      hipLaunchKernelGGL((bdf2_wide_kernel<DIAG, SP, false>), dim3(grid), dim3(kBlock), 0, p->stream, a);
    }
  }
  if (!wide)
    hipLaunchKernelGGL((bdf2_kernel<D, MT, KT, V, APART, DIAG, SP, false, ZF>), dim3(grid), dim3(SplitShape<D>::kThreads), 0,
                       p->stream, a);
  if (DIAG) hipLaunchKernelGGL(diag_finish_kernel, dim3(1), dim3(kBlock), 0, p->stream, a.part, grid, diag_out);
  return hipGetLastError();
}

// The spatial form reads FP64 velocity gradients only (an FP32-kappa plan refuses it).
template <int D, typename MT, typename KT, int V, bool APART, bool ZF>
hipError_t bdf2_go_z(const tfs_plan_s* p, const Bdf2Args<MT, KT>& a, bool diag, double* diag_out) {
  if constexpr (sizeof(KT) == 8) {
    if (a.sp.rate || a.sp.src >= 0)
      return diag ? bdf2_go_<D, MT, KT, V, APART, true, true, ZF>(p, a, diag_out)
                  : bdf2_go_<D, MT, KT, V, APART, false, true, ZF>(p, a, diag_out);
  }
  return diag ? bdf2_go_<D, MT, KT, V, APART, true, false, ZF>(p, a, diag_out)
              : bdf2_go_<D, MT, KT, V, APART, false, false, ZF>(p, a, diag_out);
}

template <int D, typename MT, typename KT, int V, bool APART>
hipError_t bdf2_go(const tfs_plan_s* p, const Bdf2Args<MT, KT>& a, bool diag, double* diag_out) {
  return p->zform ? bdf2_go_z<D, MT, KT, V, APART, true>(p, a, diag, diag_out)
                  : bdf2_go_z<D, MT, KT, V, APART, false>(p, a, diag, diag_out);
}

template <int D, typename MT, typename KT>
hipError_t bdf2_dispatch(const tfs_plan_s* p, int64_t n, const void* ka, const void* kb, const Levels& L,
                         double* tau, double* diag) {
  const int64_t st = p->stride;
  Bdf2Args<MT, KT> a;
  a.ka = static_cast<const KT*>(ka);
  a.kb = static_cast<const KT*>(kb);
  a.Xn = L.Xn;
  a.Xm = L.Xm;
  a.Xmm = p->zform ? L.Xmm : nullptr;
  a.Xo = L.Xo;
  a.Yn = static_cast<const MT*>(L.Yn);
  a.Ym = static_cast<const MT*>(L.Ym);
  a.Yo = static_cast<MT*>(L.Yo);
  a.tau = tau;
  a.coef = p->d_coef;
  a.part = L.part ? L.part : p->d_part;
  a.npoints = p->npoints;
  a.stride = st;
  a.tile = p->tile;
  a.m = p->m;
  a.s.a_diag = p->a_diag;
  a.sp.rate = p->sp_rate;
  a.sp.src = p->sp_source;
  a.s.eta = p->eta;
  a.s.s_ec = p->s_ec;
  a.s.inv_De = 1.0 / p->De;
  a.s.zeta = p->zeta[n + 1];
  a.s.tau_scale = p->tau_scale;
  const int V = pick_vec<D, MT, KT>(p, ka, kb, L, tau, 2);
  const bool dg = diag != nullptr;
  if constexpr (sizeof(MT) == 4) {
    if (V == 4) return bdf2_go<D, MT, KT, 4, false>(p, a, dg, diag);
  }
  if (V == 2) return bdf2_go<D, MT, KT, 2, false>(p, a, dg, diag);
  if (points_apart<MT>(p)) return bdf2_go<D, MT, KT, kApart<MT>, true>(p, a, dg, diag);
  return bdf2_go<D, MT, KT, 1, false>(p, a, dg, diag);
}

template <int D, typename MT, typename KT, int V, bool DIAG, bool SP>
hipError_t start_launch(const tfs_plan_s* p, StartArgs<MT, KT> a, int64_t p_begin, int64_t ngroups, int part0,
                        int* nblocks) {
  a.p_begin = p_begin;
  a.ngroups = ngroups;
  a.part0 = part0;
  const int grid = grid_for(p, ngroups);
  hipLaunchKernelGGL((start_kernel<D, MT, KT, V, DIAG, SP>), dim3(grid), dim3(kBlock), 0, p->stream, a);
  *nblocks = grid;
  return hipGetLastError();
}

template <int D, typename MT, typename KT, int V, bool DIAG, bool SP>
hipError_t start_go_(const tfs_plan_s* p, const StartArgs<MT, KT>& a, double* diag_out) {
  const int64_t full = p->npoints / V, rest = p->npoints - full * V;
  int nb = 0, nt = 0;
  hipError_t e = hipSuccess;
  if (full > 0) e = start_launch<D, MT, KT, V, DIAG, SP>(p, a, 0, full, 0, &nb);
  if (e == hipSuccess && rest > 0) e = start_launch<D, MT, KT, 1, DIAG, SP>(p, a, full * V, rest, nb, &nt);
  if (e == hipSuccess && DIAG)
    hipLaunchKernelGGL(diag_finish_kernel, dim3(1), dim3(kBlock), 0, p->stream, a.part, nb + nt, diag_out);
  return e == hipSuccess ? hipGetLastError() : e;
}

template <int D, typename MT, typename KT, int V>
hipError_t start_go(const tfs_plan_s* p, const StartArgs<MT, KT>& a, bool diag, double* diag_out) {
  if constexpr (sizeof(KT) == 8) {
    if (a.sp.rate || a.sp.src >= 0)
      return diag ? start_go_<D, MT, KT, V, true, true>(p, a, diag_out)
                  : start_go_<D, MT, KT, V, false, true>(p, a, diag_out);
  }
  return diag ? start_go_<D, MT, KT, V, true, false>(p, a, diag_out)
              : start_go_<D, MT, KT, V, false, false>(p, a, diag_out);
}

// The split step (no local solve, no diagnostics).
template <int D, typename MT, int V, bool APART>
hipError_t bdf2_split_go(const tfs_plan_s* p, Bdf2Args<MT, double> a) {
  const SplitGrid sg = split_grid(p, V);
  a.main = sg.main;
  a.wide = sg.wide;
  if constexpr (D == 2 && sizeof(MT) == 8 && !APART) {
    if (wide_step<D, MT, double>(p, V)) {
      hipLaunchKernelGGL((bdf2_wide_kernel<false, false, true>), dim3(wide_blocks(p)), dim3(kBlock), 0, p->stream, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((bdf2_kernel<D, MT, double, V, APART, false, false, true>), dim3(sg.grid),
                     dim3(SplitShape<D>::kThreads), 0, p->stream, a);
  return hipGetLastError();
}

template <int D, typename MT>
hipError_t bdf2_split_dispatch(const tfs_plan_s* p, int64_t n, const double* ka, const double* kb, const Levels& L,
                               double* G) {
  Bdf2Args<MT, double> a;
  a.ka = ka;
  a.kb = kb;
  a.Xn = L.Xn;
  a.Xm = L.Xm;
  a.Xmm = nullptr;
  a.Xo = L.Xo;
  a.Yn = static_cast<const MT*>(L.Yn);
  a.Ym = static_cast<const MT*>(L.Ym);
  a.Yo = static_cast<MT*>(L.Yo);
  a.tau = G;
  a.coef = p->d_coef;
  a.part = p->d_part;
  a.npoints = p->npoints;
  a.stride = p->stride;
  a.tile = p->tile;
  a.m = p->m;
  a.s.a_diag = p->a_diag;
  a.sp.rate = nullptr;
  a.sp.src = -1;
  a.s.eta = p->eta;
  a.s.s_ec = p->s_ec;
  a.s.inv_De = 1.0 / p->De;
  a.s.zeta = p->zeta[n + 1];
  a.s.tau_scale = p->tau_scale;
  const int V = pick_vec<D, MT, double>(p, ka, kb, L, G, 2);
  if constexpr (sizeof(MT) == 4) {
    if (V == 4) return bdf2_split_go<D, MT, 4, false>(p, a);
  }
  if (V == 2) return bdf2_split_go<D, MT, 2, false>(p, a);
  if (points_apart<MT>(p)) return bdf2_split_go<D, MT, kApart<MT>, true>(p, a);
  return bdf2_split_go<D, MT, 1, false>(p, a);
}

template <int D, typename MT, typename KT>
hipError_t start_dispatch(const tfs_plan_s* p, const void* ka, const Levels& L, double* tau, double* diag) {
  StartArgs<MT, KT> a;
  a.ka = static_cast<const KT*>(ka);
  a.X0 = L.Xn;
  a.X1 = L.Xo;
  a.Y0 = static_cast<MT*>(L.Ym0);
  a.Y1 = static_cast<MT*>(L.Yo);
  a.tau = tau;
  a.coef = p->d_coef;
  a.part = L.part ? L.part : p->d_part;
  a.stride = p->stride;
  a.tile = p->tile;
  a.m = p->m;
  a.zform = p->zform ? 1 : 0;
  a.s.hgt = p->hg * p->theta;
  a.sp.rate = p->sp_rate;
  a.sp.src = p->sp_source;
  a.s.inv_De = 1.0 / p->De;
  a.s.src1 = p->hg * p->theta;
  a.s.sigma1 = p->sigma1;
  a.s.sigma2 = p->sigma2;
  a.s.gamma = p->gamma;
  a.s.theta = p->theta;
  a.s.hr = p->hr;
  const int V = pick_vec<D, MT, KT>(p, ka, nullptr, L, tau, 2);
  const bool dg = diag != nullptr;
  if constexpr (sizeof(MT) == 4) {
    if (V == 4) return start_go<D, MT, KT, 4>(p, a, dg, diag);
  }
  if (V == 2) return start_go<D, MT, KT, 2>(p, a, dg, diag);
  return start_go<D, MT, KT, 1>(p, a, dg, diag);
}

template <int D, typename MT, typename KT, int V, bool APART, bool DIAG, bool SP>
hipError_t exp_go_(const tfs_plan_s* p, ExpArgs<MT, KT> a, double* diag_out) {
  const SplitGrid sg = split_grid(p, V);
  const int grid = sg.grid;
  a.main = sg.main;
  a.wide = sg.wide;
  a.chunked = chunked_rounds<D, MT>(p);
  hipLaunchKernelGGL((exp_kernel<D, MT, KT, V, APART, DIAG, SP>), dim3(grid), dim3(SplitShape<D>::kThreads), 0, p->stream, a);
  if (DIAG) hipLaunchKernelGGL(diag_finish_kernel, dim3(1), dim3(kBlock), 0, p->stream, a.part, grid, diag_out);
  return hipGetLastError();
}

template <int D, typename MT, typename KT, int V, bool APART, bool SP>
hipError_t exp_go_d(const tfs_plan_s* p, const ExpArgs<MT, KT>& a, double* diag) {
  return diag ? exp_go_<D, MT, KT, V, APART, true, SP>(p, a, diag) : exp_go_<D, MT, KT, V, APART, false, SP>(p, a, diag);
}

template <int D, typename MT, typename KT, bool SP>
hipError_t exp_go(const tfs_plan_s* p, const ExpArgs<MT, KT>& a, int V, double* diag) {
  if constexpr (sizeof(MT) == 4) {
    if (V == 4) return exp_go_d<D, MT, KT, 4, false, SP>(p, a, diag);
  }
  if (V == 2) return exp_go_d<D, MT, KT, 2, false, SP>(p, a, diag);
  if (points_apart<MT>(p)) return exp_go_d<D, MT, KT, kApart<MT>, true, SP>(p, a, diag);
  return exp_go_d<D, MT, KT, 1, false, SP>(p, a, diag);
}

template <int D, typename MT, typename KT>
hipError_t exp_dispatch(const tfs_plan_s* p, int64_t n, const void* ka, const void* kb, const Levels& L,
                        double* tau, double* diag) {
  ExpArgs<MT, KT> a;
  a.ka = static_cast<const KT*>(ka);
  a.kb = (n >= 1) ? static_cast<const KT*>(kb) : nullptr;
  a.Xn = L.Xn;
  a.Xo = L.Xo;
  a.Yn = static_cast<const MT*>(L.Yn);
  a.Yo = static_cast<MT*>(L.Yo);
  a.tau = tau;
  a.Hout = nullptr;
  a.coef = p->d_coef;
  a.part = L.part ? L.part : p->d_part;
  a.npoints = p->npoints;
  a.stride = p->stride;
  a.tile = p->tile;
  a.m = p->m;
  a.s.a_diag = 1.0 + p->q_e / p->De;
  a.sp.rate = p->sp_rate;
  a.sp.src = p->sp_source;
  a.s.q = p->q_e;
  a.s.s_h = p->s_h;
  a.s.inv_De = 1.0 / p->De;
  a.s.zeta = p->zeta[n + 1];
  a.s.tau_scale = p->tau_scale;
  a.s.eta_e = p->eta_e;
  a.s.fa = 1.5;
  a.s.fb = -0.5;
  a.s.first = n == 0 ? 1 : 0;
  // the level-n modes are read (not at n = 0) and written: both alignments matter
  Levels A = L;
  A.Ym = nullptr;
  const int V = pick_vec<D, MT, KT>(p, ka, a.kb, A, tau, sizeof(MT) == 4 ? 4 : 2);
  if constexpr (sizeof(KT) == 8) {
    if (a.sp.rate || a.sp.src >= 0) return exp_go<D, MT, KT, true>(p, a, V, diag);
  }
  return exp_go<D, MT, KT, false>(p, a, V, diag);
}

// The split exponential step (no local solve).
template <int D, typename MT, int V, bool APART>
hipError_t exp_split_go(const tfs_plan_s* p, ExpArgs<MT, double> a) {
  const SplitGrid sg = split_grid(p, V);
  a.main = sg.main;
  a.wide = sg.wide;
  a.chunked = chunked_rounds<D, MT>(p);
  hipLaunchKernelGGL((exp_kernel<D, MT, double, V, APART, false, false, true>), dim3(sg.grid), dim3(SplitShape<D>::kThreads),
                     0, p->stream, a);
  return hipGetLastError();
}

template <int D, typename MT>
hipError_t exp_split_dispatch(const tfs_plan_s* p, int64_t n, const double* ka, const double* kb, const Levels& L,
                              double* G, double* H) {
  ExpArgs<MT, double> a;
  a.ka = ka;
  a.kb = (n >= 1) ? kb : nullptr;
  a.Xn = L.Xn;
  a.Xo = L.Xo;
  a.Yn = static_cast<const MT*>(L.Yn);
  a.Yo = static_cast<MT*>(L.Yo);
  a.tau = G;
  a.Hout = H;
  a.coef = p->d_coef;
  a.part = nullptr;
  a.npoints = p->npoints;
  a.stride = p->stride;
  a.tile = p->tile;
  a.m = p->m;
  a.s.a_diag = 1.0 + p->q_e / p->De;
  a.sp.rate = nullptr;
  a.sp.src = -1;
  a.s.q = p->q_e;
  a.s.s_h = p->s_h;
  a.s.inv_De = 1.0 / p->De;
  a.s.zeta = p->zeta[n + 1];
  a.s.tau_scale = p->tau_scale;
  a.s.eta_e = p->eta_e;
  a.s.fa = 1.5;
  a.s.fb = -0.5;
  a.s.first = n == 0 ? 1 : 0;
  Levels A = L;
  A.Ym = nullptr;
  int V = pick_vec<D, MT, double>(p, ka, a.kb, A, G, sizeof(MT) == 4 ? 4 : 2);
  if (!aligned(H, (size_t)V * 8)) V = 1;
  if constexpr (sizeof(MT) == 4) {
    if (V == 4) return exp_split_go<D, MT, 4, false>(p, a);
  }
  if (V == 2) return exp_split_go<D, MT, 2, false>(p, a);
  if (points_apart<MT>(p)) return exp_split_go<D, MT, kApart<MT>, true>(p, a);
  return exp_split_go<D, MT, 1, false>(p, a);
}

}  // namespace

// a V-wide pass and a V = 1 tail pass
int max_blocks(const tfs_plan_s* p) { return 2 * p->num_cus * kMaxBlocksPerCU; }

// Static scratch of tfs_step_noalloc: the diagnostics block partials of one step (the V-wide
// pass and the tail pass of a 256-CU device at the default 16 blocks per CU), 384 KiB.  Every
// device holds its own copy until the process ends.  Host code never passes the symbol itself
// to a kernel or a copy: only the address scratch_address returns for the device.
static __device__ __align__(256) double scratch[(size_t)kScratchPartials * kNumDiag];

hipError_t scratch_address(int device, double** out) {
  static std::mutex mu;
  static std::vector<double*> cache;
  std::lock_guard<std::mutex> lock(mu);
  if (device < 0) return hipErrorInvalidDevice;
  if ((size_t)device < cache.size() && cache[device]) {
    *out = cache[device];
    return hipSuccess;
  }
  void* ptr = nullptr;
  const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  if ((size_t)device >= cache.size()) cache.resize((size_t)device + 1, nullptr);
  cache[device] = static_cast<double*>(ptr);
  *out = cache[device];
  return hipSuccess;
}

// The plan's (dim, mode precision, kappa precision) instance of a dispatcher; FP32 velocity
// gradients exist only with FP32 modes.
#define TFS_DISPATCH(fn, ...)                                                                      \
  (p->precision == TFS_FP64                                                                        \
       ? (p->d == 2 ? fn<2, double, double>(__VA_ARGS__) : fn<3, double, double>(__VA_ARGS__))    \
       : p->kappa_f32                                                                              \
             ? (p->d == 2 ? fn<2, float, float>(__VA_ARGS__) : fn<3, float, float>(__VA_ARGS__))  \
             : (p->d == 2 ? fn<2, float, double>(__VA_ARGS__) : fn<3, float, double>(__VA_ARGS__)))

hipError_t launch_bdf2(const tfs_plan_s* p, int64_t n, const void* ka, const void* kb, const Levels& L,
                       double* tau, double* diag) {
  if (p->npoints == 0) {
    if (diag) hipLaunchKernelGGL(diag_finish_kernel, dim3(1), dim3(kBlock), 0, p->stream, p->d_part, 0, diag);
    return hipGetLastError();
  }
  return TFS_DISPATCH(bdf2_dispatch, p, n, ka, kb, L, tau, diag);
}

hipError_t launch_bdf2_split(const tfs_plan_s* p, int64_t n, const double* ka, const double* kb, const Levels& L,
                             double* G) {
  if (p->npoints == 0) return hipSuccess;
  if (p->precision == TFS_FP64)
    return p->d == 2 ? bdf2_split_dispatch<2, double>(p, n, ka, kb, L, G)
                     : bdf2_split_dispatch<3, double>(p, n, ka, kb, L, G);
  return p->d == 2 ? bdf2_split_dispatch<2, float>(p, n, ka, kb, L, G)
                   : bdf2_split_dispatch<3, float>(p, n, ka, kb, L, G);
}

hipError_t launch_startup(const tfs_plan_s* p, const void* ka, const Levels& L, double* tau, double* diag) {
  if (p->npoints == 0) {
    if (diag) hipLaunchKernelGGL(diag_finish_kernel, dim3(1), dim3(kBlock), 0, p->stream, p->d_part, 0, diag);
    return hipGetLastError();
  }
  return TFS_DISPATCH(start_dispatch, p, ka, L, tau, diag);
}

hipError_t launch_exp(const tfs_plan_s* p, int64_t n, const void* ka, const void* kb, const Levels& L,
                      double* tau, double* diag) {
  if (p->npoints == 0) {
    if (diag) hipLaunchKernelGGL(diag_finish_kernel, dim3(1), dim3(kBlock), 0, p->stream, p->d_part, 0, diag);
    return hipGetLastError();
  }
  return TFS_DISPATCH(exp_dispatch, p, n, ka, kb, L, tau, diag);
}

hipError_t launch_exp_split(const tfs_plan_s* p, int64_t n, const double* ka, const double* kb, const Levels& L,
                            double* G, double* H) {
  if (p->npoints == 0) return hipSuccess;
  if (p->precision == TFS_FP64)
    return p->d == 2 ? exp_split_dispatch<2, double>(p, n, ka, kb, L, G, H)
                     : exp_split_dispatch<3, double>(p, n, ka, kb, L, G, H);
  return p->d == 2 ? exp_split_dispatch<2, float>(p, n, ka, kb, L, G, H)
                   : exp_split_dispatch<3, float>(p, n, ka, kb, L, G, H);
}

hipError_t launch_modes_to_plain(const tfs_plan_s* p, int64_t level, const double* X, const void* Y, double* Xk) {
  if (p->npoints == 0) return hipSuccess;
  const int64_t st = p->stride, xs = (int64_t)p->c * st;
  const double* Xs = X + (level % p->xlev) * xs;
  const double* Xm = (p->zform && level >= 1) ? X + ((level - 1) % p->xlev) * xs : nullptr;
  const int slot = p->scheme == TFS_SCHEME_EXP ? 0 : (int)(level % 2);   // the exponential scheme keeps one level
  const int64_t total = (int64_t)p->m * p->c * p->npoints;
  int grid = (int)((total + kBlock - 1) / kBlock);
  if (grid > 65536) grid = 65536;
  const int zf = p->zform ? 1 : 0;
  if (p->precision == TFS_FP64) {
    const double* Ys = static_cast<const double*>(Y) + (int64_t)slot * p->m * p->c * st;
    hipLaunchKernelGGL(plain_kernel<double>, dim3(grid), dim3(kBlock), 0, p->stream, Xs, Xm, Ys, p->d_coef, Xk,
                       p->npoints, st, p->tile, p->m, p->c, zf);
  } else {
    const float* Ys = static_cast<const float*>(Y) + (int64_t)slot * p->m * p->c * st;
    hipLaunchKernelGGL(plain_kernel<float>, dim3(grid), dim3(kBlock), 0, p->stream, Xs, Xm, Ys, p->d_coef, Xk,
                       p->npoints, st, p->tile, p->m, p->c, zf);
  }
  return hipGetLastError();
}

}  // namespace tfs
