// Shared-tree batched form: B instances of one problem (the same tree, dynamics,
// costs, boxes and risk parameters) that differ only in x0 and in their
// iterates. Every instance runs Alg. 3 (or CP) with its own decisions; the
// instances advance in lockstep rounds, one evaluation of the CP operator T
// (section 3) per round for all of them, so that the Riccati-type sweeps of
// the S1 projection (Alg. 2) see B right-hand sides per node at once: each
// per-node mat-vec of the single-instance form becomes a product of the
// node's factored matrix with a [dimension x 16 instances] tile on the
// matrix cores (MFMA 16x16x4, FP32 or FP64).
//
// Layout: vector buffers hold instance b at base + b * vs (the vector layout
// of a single problem, vs >= n_v), so the node-local passes (pre-pass,
// post-pass with the residual statistics, M) run the single-instance family
// steps on each instance. The sweep buffers q, xbar (then x) [Bp / 16][nn][nx]
// [16] and d, ubar [Bp / 16][nn][nu][16] hold a tile's 16 instances of an entry
// side by side: an MFMA operand is then 4 runs of 16 where instance-major rows
// made it 16 cache lines, which the vector memory unit takes one by one
// (both sweeps of 15 instances on 2047 nodes, FP64: 152 us against 140; 64 on 95
// nodes, FP32: 66 against 58). Bp rounds B up to 16; the extra columns run on zeros.
//
// Each instance's state machine (Alg. 3: K0, line search with K1/K2, KM), its
// Anderson ring and Gram solve (FP64) live on the device: a round is a fixed
// sequence of launches that the host queues without waiting for any of its
// results; it only polls how many instances have ended, one round behind.
#include "device_common.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <limits>
#include <vector>

namespace spk {

typedef float shf4 __attribute__((ext_vector_type(4)));
typedef double shd4 __attribute__((ext_vector_type(4)));

// One 16x16x4 step D = A B + C on a wavefront. Lane l supplies A[l % 16][l / 16]
// and B[l / 16][l % 16]; register r of lane l holds D[row(l / 16, r)][l % 16]:
// row 4 (l / 16) + r for FP32, (l / 16) + 4 r for FP64 (both measured).
template <typename S>
struct Mfma;
template <>
struct Mfma<float> {
  using acc_t = shf4;
  __device__ static acc_t step(float a, float b, acc_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int row(int kk, int r) { return 4 * kk + r; }
};
template <>
struct Mfma<double> {
  using acc_t = shd4;
  __device__ static acc_t step(double a, double b, acc_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int row(int kk, int r) { return kk + 4 * r; }
};

constexpr int kShCols = 16;   // instances per MFMA tile
static_assert(kShCols == kTileCols, "the pre-passes write tiles of this width");
constexpr int kShWaves = 16;  // wavefronts per workgroup of the sweeps

// acc += A[m0 .. m0 + 16)[0 .. nin) X, A input-major (element (out o, in k)
// at k nout + o), entry k of X's column j (instance) at x[16 k + j];
// nin <= 64. The operands of 8 steps (32 inputs) are loaded before their
// MFMAs, so a chain waits for one round of loads per 32 inputs.
template <typename S>
__device__ __forceinline__ void tile_mma(typename Mfma<S>::acc_t& acc, const S* __restrict__ A, int nout, int nin,
                                         int m0, const S* __restrict__ x, int lane) {
  const int r = lane & 15, kk = lane >> 4;
  const int m = m0 + r;
  for (int k0 = 0; k0 < nin; k0 += 32) {
    S a[8], b[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int k = k0 + 4 * t + kk;
      const bool in = k < nin;
      a[t] = (in && m < nout) ? A[(size_t)k * nout + m] : S(0);
      b[t] = in ? x[kShCols * k + r] : S(0);
    }
#pragma unroll
    for (int t = 0; t < 8; ++t)
      if (k0 + 4 * t < nin) acc = Mfma<S>::step(a[t], b[t], acc);
  }
}

template <typename S>
__device__ __forceinline__ typename Mfma<S>::acc_t zero_acc() {
  typename Mfma<S>::acc_t a;
  a[0] = a[1] = a[2] = a[3] = S(0);
  return a;
}

// ---------------------------------------------------------------- T on B instances
// pre-pass of every (unit, instance): a team of T lanes per family or leaf
// (flat_pre_family; q = -xbar at a leaf). IX: 32-bit offsets while one
// instance's iterate and the node arrays stay below 4 GiB.
template <typename S, int T, int SL, typename IX>
__global__ void __launch_bounds__(256) k_sh_pre(DevProb<S> P, const S* __restrict__ v, S* __restrict__ Tv,
                                                S* __restrict__ xbar, S* __restrict__ ubar, S* __restrict__ q,
                                                long long vs) {
  const int lane = threadIdx.x % T;
  const int i = blockIdx.x * (256 / T) + threadIdx.x / T;
  if (i >= P.nn) return;  // whole teams only; no block barrier below
  const size_t b = blockIdx.y;
  const int nx = P.nx, nu = P.nu;
  const Off<S, IX> O(P);
  const S* z = v + b * vs;
  const S* eta = z + P.nz;
  S* const qb = q + tile_base(b, (size_t)P.nn * nx);
  if (i >= P.nl) {
    for (int o = lane; o < nx; o += T) {
      const IX e3 = O.e3(i) + o;
      const S Lt = at<S, IX>(eta, e3) + at<S, IX>(P.sqN, (IX)i * nx + o) * at<S, IX>(eta, e3 + nx);
      qb[((size_t)i * nx + o) * kShCols] = P.alpha * Lt - at<S, IX>(z, O.x(i) + o);
    }
    return;
  }
  S bar[SL];
  flat_pre_family<S, T, SL, IX>(P, O, z, eta, Tv + b * vs, i, P.fc[i], P.nch[i], lane, bar);
#pragma unroll
  for (int k = 0; k < SL; ++k) {
    const int o = lane + T * k;
    if (o < nx) xbar[tile_base(b, (size_t)P.nn * nx) + ((size_t)i * nx + o) * kShCols] = bar[k];
    else if (o < nx + nu) ubar[tile_base(b, (size_t)P.nn * nu) + ((size_t)i * nu + (o - nx)) * kShCols] = bar[k];
  }
}

// The sweeps of Alg. 2 for 16 instances per workgroup, workgroup barriers
// between stages. The work of a stage is split into (node, 16-row tile)
// items spread over the wavefronts: backward, the tiles of d^i and of q^i
// (independent given the children's q); forward, the tiles of u^i and of
// every child's x^c (independent given x^i and d^i). Backward (one mat-vec
// phase): d^i = R~^{-1} ubar^i + sum_c Bt^c q^c, q^i = P1 ubar^i - xbar^i +
// sum_c At^c q^c. Forward: u^i = K x^i + d^i, x^c = Abar^c x^i + B^c d^i.
//
// The stages are cut into segments [ta, tb): the subtrees rooted at stage ta
// are independent down to stage tb - 1, so a launch runs one workgroup per
// (tile group, node of stage ta) over its part of the segment, bottom-up
// (backward) or top-down (forward); the segments run in order, so that the
// wide stages spread over the compute units. A tree of one segment runs both
// sweeps in one launch.
//
// The host learns one round late that every instance has ended, so a round may
// be queued that nobody needs: its sweeps end at once when *count (instances
// that have ended) reaches all. One wavefront reads the count while another
// finds the node ranges, so that the check adds nothing to a launch (read by
// every wavefront it took 0.2 us of 14).
struct ShDone {
  const unsigned* count;
  unsigned all;
};
constexpr int kShMaxLevels = 128;  // stages of a segment a workgroup keeps in LDS

struct ShSweepArgs {
  int maxch, ta, tb, nsub;  // nsub: nodes of stage ta (subtrees per tile group)
};

template <typename S>
__device__ __forceinline__ void sh_bwd_nodes(const DevProb<S>& P, int i0, int i1, S* q0, S* d0, const S* xb0,
                                             const S* ub0, int lane, int wave) {
  using acc_t = typename Mfma<S>::acc_t;
  const int col = lane & 15, kk = lane >> 4;
  const int nx = P.nx, nu = P.nu;
  const int tu = (nu + 15) / 16, tx = (nx + 15) / 16;
  const int items = (i1 - i0) * (tu + tx);
  for (int it = wave; it < items; it += kShWaves) {
    const int i = i0 + it / (tu + tx), sub = it % (tu + tx);
    const int fc = P.fc[i], n = P.nch[i];
    acc_t acc = zero_acc<S>();
    if (sub < tu) {  // d^i, rows 16 sub ..
      const int m0 = 16 * sub;
      tile_mma<S>(acc, P.Rinv + (size_t)i * nu * nu, nu, nu, m0, ub0 + (size_t)i * nu * kShCols, lane);
      for (int k = 0; k < n; ++k)
        tile_mma<S>(acc, P.BtR + (size_t)(fc + k) * nx * nu, nu, nx, m0, q0 + (size_t)(fc + k) * nx * kShCols, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + Mfma<S>::row(kk, r);
        if (m < nu) d0[((size_t)i * nu + m) * kShCols + col] = acc[r];
      }
    } else {  // q^i
      const int m0 = 16 * (sub - tu);
      tile_mma<S>(acc, P.P1C + (size_t)i * nu * nx, nx, nu, m0, ub0 + (size_t)i * nu * kShCols, lane);
      for (int k = 0; k < n; ++k)
        tile_mma<S>(acc, P.AtR + (size_t)(fc + k) * nx * nx, nx, nx, m0, q0 + (size_t)(fc + k) * nx * kShCols, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + Mfma<S>::row(kk, r);
        if (m < nx) {
          const size_t e = ((size_t)i * nx + m) * kShCols + col;
          q0[e] = acc[r] - xb0[e];
        }
      }
    }
  }
}

template <typename S>
__device__ __forceinline__ void sh_fwd_nodes(const DevProb<S>& P, int i0, int i1, S* z0, S* xt0, const S* d0,
                                             long long vs, int maxch, int lane, int wave) {
  using acc_t = typename Mfma<S>::acc_t;
  const int col = lane & 15, kk = lane >> 4;
  const int nx = P.nx, nu = P.nu;
  const int tu = (nu + 15) / 16, tx = (nx + 15) / 16;
  const Off<S> O(P);
  const int per = tu + maxch * tx;
  const int items = (i1 - i0) * per;
  for (int it = wave; it < items; it += kShWaves) {
    const int i = i0 + it / per, sub = it % per;
    const int fc = P.fc[i], n = P.nch[i];
    const S* xi = xt0 + (size_t)i * nx * kShCols;
    const S* di = d0 + (size_t)i * nu * kShCols;
    acc_t acc = zero_acc<S>();
    if (sub < tu) {  // u^i
      const int m0 = 16 * sub;
      tile_mma<S>(acc, P.KC + (size_t)i * nx * nu, nu, nx, m0, xi, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + Mfma<S>::row(kk, r);
        if (m < nu) z0[(size_t)col * vs + O.u(i) + m] = acc[r] + di[m * kShCols + col];
      }
    } else {  // x^c of child k
      const int k = (sub - tu) / tx, m0 = 16 * ((sub - tu) % tx);
      if (k >= n) continue;
      const int c = fc + k;
      tile_mma<S>(acc, P.AbC + (size_t)c * nx * nx, nx, nx, m0, xi, lane);
      tile_mma<S>(acc, P.BC + (size_t)c * nu * nx, nx, nu, m0, di, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + Mfma<S>::row(kk, r);
        if (m < nx) {
          z0[(size_t)col * vs + O.x(c) + m] = acc[r];
          if (c < P.nl) xt0[((size_t)c * nx + m) * kShCols + col] = acc[r];
        }
      }
    }
  }
}

// DIR: 1 backward, 2 forward, 3 both (builds of their own: one that can do both,
// told at run time, took 0.4 us a launch more)
template <typename S, int DIR>
__global__ void __launch_bounds__(64 * kShWaves) k_sh_sweeps(DevProb<S> P, const int* __restrict__ stage_off,
                                                              S* __restrict__ Tv, const double* __restrict__ x0s,
                                                              S* __restrict__ xbar, S* __restrict__ ubar,
                                                              S* __restrict__ q, S* __restrict__ d, long long vs,
                                                              ShSweepArgs A, ShDone done) {
  __shared__ int lo[kShMaxLevels], hi[kShMaxLevels];
  __shared__ unsigned ended;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = blockIdx.x / A.nsub, r = blockIdx.x % A.nsub;  // tile group, subtree
  const size_t b0 = (size_t)g * kShCols;
  const int nx = P.nx, nu = P.nu;
  const size_t wx = (size_t)P.nn * nx, wu = (size_t)P.nn * nu;
  const Off<S> O(P);
  S* q0 = q + b0 * wx;
  S* d0 = d + b0 * wu;
  S* xb0 = xbar + b0 * wx;  // xbar in the backward sweep, then x in the forward one
  S* z0 = Tv + b0 * vs;
  // node ranges of the subtree rooted at node stage_off[ta] + r, per stage
  const int levels = A.tb - A.ta;
  if (threadIdx.x == 64) ended = *done.count;
  if (threadIdx.x == 0) {
    lo[0] = stage_off[A.ta] + r;
    hi[0] = lo[0] + 1;
    for (int l = 1; l < levels; ++l) {
      lo[l] = P.fc[lo[l - 1]];
      hi[l] = P.fc[hi[l - 1] - 1] + P.nch[hi[l - 1] - 1];
    }
  }
  auto root = [&]() {  // root state of every instance, in xbar's place
    for (int e = threadIdx.x; e < kShCols * nx; e += blockDim.x) {
      const int j = e / nx, o = e % nx;
      const S x = (S)x0s[(b0 + j) * nx + o];
      z0[(size_t)j * vs + O.x(0) + o] = x;
      xb0[(size_t)o * kShCols + j] = x;
    }
  };
  if (DIR == 2 && A.ta == 0) root();
  __syncthreads();
  if (ended >= done.all) return;
  if (DIR & 1) {
    for (int l = levels - 1; l >= 0; --l) {
      sh_bwd_nodes<S>(P, lo[l], hi[l], q0, d0, xb0, ubar + b0 * wu, lane, wave);
      __syncthreads();
    }
  }
  if (DIR == 3) {
    root();
    __syncthreads();
  }
  if (DIR & 2) {
    for (int l = 0; l < levels; ++l) {
      sh_fwd_nodes<S>(P, lo[l], hi[l], z0, xb0, d0, vs, A.maxch, lane, wave);
      __syncthreads();
    }
  }
}

// post-pass of every (unit, instance): dual update and the instance's residual
// statistics (block records at partials + b * gridDim.x * kStats)
template <typename S, int T, int SL, typename IX>
__global__ void __launch_bounds__(256) k_sh_post(DevProb<S> P, const long long* __restrict__ spos,
                                                 const S* __restrict__ v, S* __restrict__ Tv, long long vs,
                                                 double* __restrict__ partials) {
  const int lane = threadIdx.x % T;
  const int i = blockIdx.x * (256 / T) + threadIdx.x / T;
  const size_t b = blockIdx.y;
  const S* z = v + b * vs;
  const S* eta = z + P.nz;
  S* zo = Tv + b * vs;
  S* eo = zo + P.nz;
  const Off<S, IX> O(P);
  StatAcc st;
  if (i < P.nl) {
    const IX xi = O.x(i), ui = O.u(i);
    flat_family<S, T, SL, IX>(P, O, (IX)spos[i], z, eta, zo, eo, i, P.fc[i], P.nch[i], lane,
                              [&](int k) { return at<S, IX>(zo, k < P.nx ? xi + k : ui + (k - P.nx)); }, st);
  } else if (i < P.nn) {
    const IX xj = O.x(i);
    flat_leaf<S, T, SL, IX>(P, O, (IX)spos[i], z, eta, zo, eo, i, lane, [&](int k) { return at<S, IX>(zo, xj + k); },
                            st);
  }
  const double w[kStats] = {team_sum<64>(st.rz2), team_sum<64>(st.re2), team_sum<64>(st.cross), wave_max(st.xip),
                            wave_max(st.xid)};
  __shared__ double red[4][kStats];
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int k = 0; k < kStats; ++k) red[threadIdx.x >> 6][k] = w[k];
  __syncthreads();
  if (threadIdx.x < kStats) {
    const int k = threadIdx.x;
    double a = red[0][k];
    for (int j = 1; j < 4; ++j) a = (k < 3) ? a + red[j][k] : fmax(a, red[j][k]);
    partials[(b * gridDim.x + blockIdx.x) * kStats + k] = a;
  }
}

// ---------------------------------------------------------------- vector steps
// Buffers of the engine, each [Bp][vs], one copy per instance (accepted points
// are copied, since instances decide differently in one round).
template <typename S>
struct ShVec {
  S* v;     // iterate
  S* tv;    // T(v)
  S* rcur;  // residual v - T(v)
  S* dir;   // direction
  S* md;    // M dir
  S* vt;    // point of the next evaluation
  S* tvt;   // T(vt)
  S* E;     // Anderson columns dV - dR, slot s at E + s * Bp * vs
  S* R;     // Anderson columns dR, slot s at R + s * Bp * vs
  long long vs, nv, slot;  // instance stride, vector length, slot stride
};

// State of one instance (device). Alg. 3 in phases: the phase says what the
// evaluation of T that has just run was for.
enum ShPhase : int { kShInit, kShK0, kShLS, kShK2, kShKM, kShCP, kShDone };
enum ShNext : int { kShHold, kShDir, kShCombo, kShTv, kShFinish };
struct ShState {
  int phase, status, k, ls, t_evals, n_k0, n_k1, n_k2, n_km, n_bt;
  int commit;  // of this round: 0 nothing, 1 v = vt, 2 also the Anderson push
  int prep;    // a residual and a direction follow the commit
  int next;    // what the next evaluation's point is formed from (ShNext)
  int line;    // the direction opens a line search: d is stored and M d formed
  double xi0, xi, om2, tol, zeta, omega_safe, omega, tau;
  double coef[5];  // kShCombo: of v, dir, vt, T(vt), r
  double s0;       // s^0 of the returned point
  AARingDev ring;
  AAPush push;
  double G[kAAMax * kAAMax], gamma[kAAMax];
};
struct ShSettings {
  double eps_abs, eps_rel, c0, c1, c2, beta, sigma, lambda;
  int max_iters, max_ls, m, cp;
};
// Buffers of the caller, one entry per instance
template <typename S>
struct ShIO {
  const double* x0;
  S* vio;
};
// What the host polls (pinned): rounds finished and instances ended
struct ShMail {
  unsigned long long round, done;
};

// Inputs of every instance in one launch: the warm start into vt, x0 into x0s,
// the box test and the initial state (padding and rejected instances run on
// zeros).
template <typename S>
__global__ void __launch_bounds__(256) k_sh_load(ShVec<S> V, const ShIO<S>* __restrict__ io, int B, int nx, int m,
                                                 const double* __restrict__ box, double* __restrict__ x0s,
                                                 ShState* __restrict__ state, unsigned* __restrict__ done) {
  const int b = blockIdx.y;
  bool out = false;
  if (b < B && (int)threadIdx.x < nx) {
    const double x = io[b].x0[threadIdx.x];
    out = !(x >= box[threadIdx.x] && x <= box[nx + threadIdx.x]);
    if (blockIdx.x == 0) x0s[(size_t)b * nx + threadIdx.x] = x;
  } else if (blockIdx.x == 0 && (int)threadIdx.x < nx) {
    x0s[(size_t)b * nx + threadIdx.x] = 0.0;
  }
  const bool rejected = __syncthreads_or(out);
  const bool on = b < B && !rejected;
  S* vt = V.vt + (size_t)b * V.vs;
  for (long long e = blockIdx.x * 256LL + threadIdx.x; e < V.nv; e += gridDim.x * 256LL) vt[e] = on ? io[b].vio[e] : S(0);
  if (blockIdx.x == 0 && threadIdx.x == 0 && b < B) {
    ShState s{};
    s.phase = on ? kShInit : kShDone;
    s.status = on ? 0 : SPOCK_REJECTED;
    s.tau = 1.0;
    s.ring.m = m;
    state[b] = s;
    if (!on) atomicAdd(done, 1u);
  }
}

// <vt - T(vt), M d> of the instances in a line search: block records in fixed
// ranges (the decision adds them in order)
template <typename S>
__global__ void __launch_bounds__(256) k_sh_rdot(ShVec<S> V, const ShState* __restrict__ state, double* __restrict__ part) {
  const size_t b = blockIdx.y;
  if (state[b].phase != kShLS) return;
  const size_t o = b * V.vs;
  double acc = 0;
  for (long long e = blockIdx.x * 256LL + threadIdx.x; e < V.nv; e += gridDim.x * 256LL)
    acc += ((double)V.vt[o + e] - (double)V.tvt[o + e]) * (double)V.md[o + e];
  acc = team_sum<64>(acc);
  __shared__ double red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) part[b * gridDim.x + blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// Per-instance sums of K values over n records (ld doubles apart), the last
// two as maxima when MAX: threads stride over the records, then wavefronts in
// order; results in every thread of the workgroup (256 threads).
template <int K, bool MAX>
__device__ __forceinline__ void sh_records(const double* __restrict__ rec, int n, int ld, double (&v)[K],
                                           double (*red)[4]) {
  constexpr int ks = MAX ? K - 2 : K;
#pragma unroll
  for (int j = 0; j < K; ++j) v[j] = 0;
  for (int r = threadIdx.x; r < n; r += 256)
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const double x = rec[(size_t)r * ld + j];
      v[j] = j < ks ? v[j] + x : fmax(v[j], x);
    }
#pragma unroll
  for (int j = 0; j < K; ++j) {
    v[j] = j < ks ? team_sum<64>(v[j]) : wave_max(v[j]);
    if ((threadIdx.x & 63) == 0) red[j][threadIdx.x >> 6] = v[j];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < K; ++j) {
    double a = red[j][0];
    for (int w = 1; w < 4; ++w) a = j < ks ? a + red[j][w] : fmax(a, red[j][w]);
    v[j] = a;
  }
  __syncthreads();
}

// First half of an instance's decisions, from the statistics of the evaluation
// that has just run: accept it (the commit and what follows) or form another
// point (K2, a shorter step, KM).
__global__ void __launch_bounds__(256) k_sh_judge(ShState* __restrict__ state, ShSettings s, const double* __restrict__ stats,
                                                  int nstat, const double* __restrict__ rdots, int nrd, double alpha,
                                                  unsigned* __restrict__ done) {
  __shared__ double red[kStats][4];
  const int b = blockIdx.x;
  ShState& I = state[b];
  const int phase = I.phase;
  if (phase == kShDone) {
    if (threadIdx.x == 0) {
      I.commit = I.prep = 0;
      I.next = kShHold;
      I.line = 0;
    }
    return;
  }
  double v[kStats], rd[1] = {0};
  sh_records<kStats, true>(stats + (size_t)b * nstat * kStats, nstat, kStats, v, red);
  if (phase == kShLS) sh_records<1, false>(rdots + (size_t)b * nrd, nrd, 1, rd, red);
  if (threadIdx.x != 0) return;
  const double om2 = v[0] + v[1] - 2.0 * alpha * v[2], xi = fmax(v[3], v[4]);
  const double om = sqrt(fmax(om2, 0.0));
  const bool ok = isfinite(v[3]) && isfinite(v[4]) && isfinite(om2);
  I.t_evals++;
  I.commit = I.prep = 0;
  I.next = kShHold;
  I.line = 0;
  auto accept = [&](int mode) {
    I.commit = mode;
    I.xi = xi;
    I.om2 = om2;
    if (!ok) {
      I.phase = kShDone;  // T of the point reached is returned
      I.status = SPOCK_NUMERICAL;
      I.next = kShFinish;
      atomicAdd(done, 1u);
    } else {
      I.prep = 1;
      if (mode == 2) I.push = aa_next_push(&I.ring);
    }
  };
  if (phase == kShInit) {
    I.xi0 = xi;
    I.tol = fmax(s.eps_abs, s.eps_rel * xi);
    I.zeta = I.omega_safe = om;
    accept(1);
  } else if (phase == kShCP) {
    I.k++;
    accept(1);
  } else if (phase != kShLS) {  // K0, K2, KM
    I.k++;
    accept(2);
  } else {
    bool backtrack = !ok;
    if (ok) {
      if (om == 0.0 || (I.omega <= I.omega_safe && om <= s.c1 * I.omega)) {  // K1
        I.omega_safe = om + pow(s.c2, (double)I.k);
        I.n_k1++;
        I.k++;
        accept(2);
      } else {
        const double rho = om * om - I.tau * rd[0];
        if (rho >= s.sigma * om * I.omega) {  // K2: v - c (vt - T vt)
          const double c = s.lambda * rho / (om * om);
          I.next = kShCombo;
          I.coef[0] = 1.0;
          I.coef[1] = 0.0;
          I.coef[2] = -c;
          I.coef[3] = c;
          I.coef[4] = 0.0;
          I.n_k2++;
          I.phase = kShK2;
        } else {
          backtrack = true;
        }
      }
    }
    if (backtrack) {
      I.tau *= s.beta;
      I.n_bt++;
      const bool again = ++I.ls < s.max_ls;
      I.next = kShCombo;
      I.coef[0] = 1.0;
      I.coef[1] = again ? I.tau : 0.0;
      I.coef[2] = I.coef[3] = 0.0;
      I.coef[4] = again ? 0.0 : -s.lambda;  // the plain KM step
      if (!again) {
        I.n_km++;
        I.phase = kShKM;
      }
    }
  }
}

// Accepting the evaluated point, in one pass: r = vt - T(vt); with commit 2 the
// Anderson push against the iterate it replaces (dR = r - r_old, E = (vt - v)
// - dR into the push's slot) and the block sums of <dR_j, dR>, <dR, dR>,
// <dR_j, r>, <dR, r> (columns oldest first); then v = vt, T(v) = T(vt). Bound by
// its traffic (4 + columns vectors read, 5 written); as a copy of four vectors
// and a push of one workgroup per instance it took 42 + 537 us for 15 instances
// of the 2047-node tree in FP64.
template <typename S>
__global__ void __launch_bounds__(256) k_sh_commit(ShVec<S> V, const ShState* __restrict__ state, int cp,
                                                   double* __restrict__ part) {
  const size_t b = blockIdx.y;
  const ShState& I = state[b];
  const int mode = I.commit;
  if (mode == 0) return;
  const size_t o = b * V.vs;
  const S* vt = V.vt + o;
  const S* tvt = V.tvt + o;
  S* v = V.v + o;
  S* tv = V.tv + o;
  S* rc = V.rcur + o;
  const long long e0 = blockIdx.x * 256LL + threadIdx.x, de = gridDim.x * 256LL;
  if (mode == 1 || cp) {
    for (long long e = e0; e < V.nv; e += de) {
      const S x = vt[e], t = tvt[e];
      v[e] = x;
      tv[e] = t;
      if (!cp) rc[e] = (S)((double)x - (double)t);
    }
    return;
  }
  const AAPush a = I.push;
  const S* Rj[kAAMax - 1];
#pragma unroll
  for (int j = 0; j < kAAMax - 1; ++j) Rj[j] = V.R + (size_t)(j < a.mo ? a.order_old[j] : 0) * V.slot + o;
  S* En = V.E + (size_t)a.slot * V.slot + o;
  S* Rn = V.R + (size_t)a.slot * V.slot + o;
  double acc[2 * kAAMax];
#pragma unroll
  for (int j = 0; j < 2 * kAAMax; ++j) acc[j] = 0;
  for (long long e = e0; e < V.nv; e += de) {
    const S x = vt[e], t = tvt[e], vo = v[e], ro = rc[e];
    S col[kAAMax - 1];
#pragma unroll
    for (int j = 0; j < kAAMax - 1; ++j) col[j] = j < a.mo ? Rj[j][e] : S(0);
    const S r = x - t, dr = r - ro;
    v[e] = x;
    tv[e] = t;
    rc[e] = r;
    Rn[e] = dr;
    En[e] = (S)(((double)x - (double)vo) - (double)dr);
#pragma unroll
    for (int j = 0; j < kAAMax - 1; ++j) {
      acc[j] += (double)col[j] * (double)dr;
      acc[kAAMax + j] += (double)col[j] * (double)r;
    }
    acc[kAAMax - 1] += (double)dr * (double)dr;
    acc[2 * kAAMax - 1] += (double)dr * (double)r;
  }
  __shared__ double red[4][2 * kAAMax];
#pragma unroll
  for (int j = 0; j < 2 * kAAMax; ++j) {
    acc[j] = team_sum<64>(acc[j]);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][j] = acc[j];
  }
  __syncthreads();
  if (threadIdx.x < 2 * kAAMax) {
    const int j = threadIdx.x;
    part[(b * gridDim.x + blockIdx.x) * (2 * kAAMax) + j] = ((red[0][j] + red[1][j]) + red[2][j]) + red[3][j];
  }
}

// The Gram solve with MO older columns from the summed dot products
template <int MO>
__device__ __noinline__ void sh_gram(ShState& I, const double (&d)[2 * kAAMax]) {
  double dots[8], Gold[16];
#pragma unroll
  for (int j = 0; j < 8; ++j) dots[j] = 0;
#pragma unroll
  for (int j = 0; j < MO; ++j) {
    dots[j] = d[j];
    dots[MO + 1 + j] = d[kAAMax + j];
  }
  dots[MO] = d[kAAMax - 1];
  dots[2 * MO + 1] = d[2 * kAAMax - 1];
  const AAPush a = I.push;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) Gold[i * 4 + j] = (i < MO && j < MO) ? I.G[a.order_old[i] * a.m + a.order_old[j]] : 0.0;
  aa_solve_dev<MO>(I.G, dots, Gold, a, I.gamma, &I.ring);
}

// Second half: the Gram solve, then the top of the next iteration of Alg. 3.
__global__ void __launch_bounds__(256) k_sh_plan(ShState* __restrict__ state, ShSettings s, const double* __restrict__ part,
                                                 int npart, unsigned* __restrict__ done) {
  __shared__ double red[2 * kAAMax][4];
  const int b = blockIdx.x;
  ShState& I = state[b];
  if (!I.prep) return;
  const bool push = I.commit == 2 && !s.cp;
  double d[2 * kAAMax];
  if (push) sh_records<2 * kAAMax, false>(part + (size_t)b * npart * (2 * kAAMax), npart, 2 * kAAMax, d, red);
  if (threadIdx.x != 0) return;
  if (push) {
    switch (I.push.mo) {
      case 0: sh_gram<0>(I, d); break;
      case 1: sh_gram<1>(I, d); break;
      case 2: sh_gram<2>(I, d); break;
      default: sh_gram<3>(I, d); break;
    }
  } else {
    I.ring.dk = 0;
  }
  if (I.xi <= I.tol || I.k >= s.max_iters) {
    I.status = I.xi <= I.tol ? SPOCK_CONVERGED : SPOCK_MAXITER;
    I.phase = kShDone;
    I.next = kShFinish;
    atomicAdd(done, 1u);
    return;
  }
  if (s.cp) {
    I.phase = kShCP;
    I.next = kShTv;
    return;
  }
  I.omega = sqrt(fmax(I.om2, 0.0));
  I.next = kShDir;
  if (I.omega <= s.c0 * I.zeta) {  // K0: v + d
    I.zeta = I.omega;
    I.n_k0++;
    I.phase = kShK0;
    return;
  }
  I.line = 1;  // the line search from tau = 1
  I.tau = 1.0;
  I.ls = 0;
  I.phase = kShLS;
}

// The point of the next evaluation: v + d with d = -r - sum_j gamma_j E_j (d
// stored when a line search opens), a combination of v, d, vt, T(vt), r, or
// T(v) (CP); or the returned point T(v) of an instance that ended. Block (0, 0)
// publishes the round and how many instances have ended.
template <typename S>
__global__ void __launch_bounds__(256) k_sh_next(ShVec<S> V, ShState* __restrict__ state, int B, const ShIO<S>* __restrict__ io,
                                                 const unsigned* __restrict__ done, ShMail* mail, unsigned long long round) {
  const size_t b = blockIdx.y;
  if (blockIdx.x == 0 && b == 0 && threadIdx.x == 0) {
    __hip_atomic_store(&mail->done, (unsigned long long)*done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&mail->round, round, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  if ((int)b >= B) return;
  const ShState& I = state[b];
  const int next = I.next;
  if (next == kShHold) return;
  const size_t o = b * V.vs;
  const S* v = V.v + o;
  const S* tv = V.tv + o;
  S* vt = V.vt + o;
  const long long e0 = blockIdx.x * 256LL + threadIdx.x, de = gridDim.x * 256LL;
  if (next == kShDir) {
    const int dk = I.ring.dk, line = I.line;
    double g[kAAMax];
    const S* E[kAAMax];
#pragma unroll
    for (int j = 0; j < kAAMax; ++j) {
      g[j] = j < dk ? I.gamma[j] : 0.0;
      E[j] = V.E + (size_t)(j < dk ? I.ring.dslot[j] : 0) * V.slot + o;
    }
    const S* r = V.rcur + o;
    S* dir = V.dir + o;
    for (long long e = e0; e < V.nv; e += de) {
      double acc = -(double)r[e];
      S c[kAAMax];
#pragma unroll
      for (int j = 0; j < kAAMax; ++j) c[j] = j < dk ? E[j][e] : S(0);
#pragma unroll
      for (int j = 0; j < kAAMax; ++j) acc -= g[j] * (double)c[j];
      if (line) {
        const S q = (S)acc;
        dir[e] = q;
        acc = (double)q;
      }
      vt[e] = (S)((double)v[e] + acc);
    }
  } else if (next == kShCombo) {
    const double c0 = I.coef[0], c1 = I.coef[1], c2 = I.coef[2], c3 = I.coef[3], c4 = I.coef[4];
    const S* dir = V.dir + o;
    const S* tvt = V.tvt + o;
    const S* r = V.rcur + o;
    for (long long e = e0; e < V.nv; e += de) {
      double acc = c0 * (double)v[e];
      if (c1 != 0.0) acc += c1 * (double)dir[e];
      if (c2 != 0.0) acc += c2 * (double)vt[e];
      if (c3 != 0.0) acc += c3 * (double)tvt[e];
      if (c4 != 0.0) acc += c4 * (double)r[e];
      vt[e] = (S)acc;
    }
  } else if (next == kShTv) {
    for (long long e = e0; e < V.nv; e += de) vt[e] = tv[e];
  } else {
    S* out = io[b].vio;
    for (long long e = e0; e < V.nv; e += de) out[e] = tv[e];
    if (e0 == 0) state[b].s0 = (double)tv[0];
  }
}

// md = M dir of the instances whose line search opens, one team of T lanes per family
template <typename S, int T>
__global__ void __launch_bounds__(256) k_sh_M(DevProb<S> P, ShVec<S> V, const ShState* __restrict__ state) {
  const size_t b = blockIdx.y;
  if (!state[b].line) return;
  const int lane = threadIdx.x % T;
  const int i = blockIdx.x * (blockDim.x / T) + threadIdx.x / T;
  if (i >= P.nl) return;
  fam_apply_M<S, T>(P, V.dir + b * V.vs, V.md + b * V.vs, i, lane);
}

// ---------------------------------------------------------------- host engine
namespace {

// Device workspace of the engine (kept between calls, not thread safe).
struct ShCache {
  void* mem = nullptr;
  size_t bytes = 0;
  void* host = nullptr;  // pinned: the mail, then the tables up and the states down
  size_t host_bytes = 0;
};
ShCache& sh_cache() {
  static ShCache c;
  return c;
}

template <typename S>
const DevProb<S>& sh_dev(const Problem& P);
template <>
const DevProb<double>& sh_dev<double>(const Problem& P) { return P.dp64; }
template <>
const DevProb<float>& sh_dev<float>(const Problem& P) { return P.dp32; }

#define SH_TRY(x)                             \
  do {                                        \
    if ((x) != hipSuccess) return SPOCK_EHIP; \
  } while (0)

// Lanes per unit of the flat passes: the fewest that hold a state and an input
int sh_team(const Problem& P) {
  int t = 8;
  while (t < P.nx + P.nu && t < 64) t <<= 1;
  return t;
}
// 32-bit offsets: one instance's iterate and the node arrays below 4 GiB
template <typename S>
bool sh_narrow(const Problem& P) {
  const unsigned long long lim = (1ull << 32) / sizeof(S);
  return (unsigned long long)(P.nz + P.neta) < lim &&
         (unsigned long long)P.tree->nn * (8ull * P.nx + 8ull * P.nu) < lim;
}
int sh_post_blocks(const Problem& P) {
  const int tpb = 256 / sh_team(P);
  return (P.tree->nn + tpb - 1) / tpb;
}

template <typename S>
hipError_t sh_launch_pre(const Problem& P, const DevProb<S>& D, const S* in, S* out, S* xbar, S* ubar, S* q,
                         long long vs, int Bp, hipStream_t st) {
  const dim3 grid(sh_post_blocks(P), Bp);
  auto go = [&](auto k) { hipLaunchKernelGGL(k, grid, dim3(256), 0, st, D, in, out, xbar, ubar, q, vs); };
  const bool nar = sh_narrow<S>(P);
  switch (sh_team(P)) {
    case 8: nar ? go(k_sh_pre<S, 8, 1, unsigned>) : go(k_sh_pre<S, 8, 1, long long>); break;
    case 16: nar ? go(k_sh_pre<S, 16, 1, unsigned>) : go(k_sh_pre<S, 16, 1, long long>); break;
    case 32: nar ? go(k_sh_pre<S, 32, 1, unsigned>) : go(k_sh_pre<S, 32, 1, long long>); break;
    default:
      if (P.nx + P.nu <= 64) nar ? go(k_sh_pre<S, 64, 1, unsigned>) : go(k_sh_pre<S, 64, 1, long long>);
      else nar ? go(k_sh_pre<S, 64, 2, unsigned>) : go(k_sh_pre<S, 64, 2, long long>);
      break;
  }
  return hipGetLastError();
}

template <typename S>
hipError_t sh_launch_post(const Problem& P, const DevProb<S>& D, const S* v, S* Tv, long long vs, double* partials,
                          int Bp, hipStream_t st) {
  const dim3 grid(sh_post_blocks(P), Bp);
  auto go = [&](auto k) { hipLaunchKernelGGL(k, grid, dim3(256), 0, st, D, P.d_spos, v, Tv, vs, partials); };
  const bool nar = sh_narrow<S>(P);
  switch (sh_team(P)) {
    case 8: nar ? go(k_sh_post<S, 8, 1, unsigned>) : go(k_sh_post<S, 8, 1, long long>); break;
    case 16: nar ? go(k_sh_post<S, 16, 1, unsigned>) : go(k_sh_post<S, 16, 1, long long>); break;
    case 32: nar ? go(k_sh_post<S, 32, 1, unsigned>) : go(k_sh_post<S, 32, 1, long long>); break;
    default:
      if (P.nx + P.nu <= 64) nar ? go(k_sh_post<S, 64, 1, unsigned>) : go(k_sh_post<S, 64, 1, long long>);
      else nar ? go(k_sh_post<S, 64, 2, unsigned>) : go(k_sh_post<S, 64, 2, long long>);
      break;
  }
  return hipGetLastError();
}

// Segments of stages of the sweeps: cut[k] .. cut[k + 1] - 1. A segment grows
// while the items of its widest stage (nodes of one subtree times the 16-row
// tiles of d and q) have a wavefront each, so chains
// and narrow stages stay in one launch and a wide stage is spread over one
// workgroup per subtree. 2047-node binary tree, n_x = n_u = 20, 15 instances,
// FP64: both sweeps 140 us in 8 launches (four segments) against 680 us in the 4
// launches of one cut at stage 3 (8 workgroups below it); the 95-node tree
// keeps its cut at stage 3. SPOCK_SH_CUT sets one cut instead (0: one launch
// over the whole tree).
struct ShPlan {
  std::vector<int> cut;
  int maxch = 1;
};
ShPlan sh_plan(const Problem& P) {
  const Tree& Tr = *P.tree;
  ShPlan L;
  for (int i = 0; i < Tr.nl; ++i) L.maxch = std::max(L.maxch, Tr.nch[i]);
  L.cut.push_back(0);
  if (const char* env = std::getenv("SPOCK_SH_CUT")) {
    const int c = std::atoi(env);
    if (c >= 1 && c < Tr.N) L.cut.push_back(c);
  } else {
    const int tiles = (P.nx + 15) / 16 + (P.nu + 15) / 16;
    // node ranges of stage t under every node of the segment's first stage
    std::vector<int> lo(1, 0), hi(1, 1);
    for (int t = 1; t < Tr.N; ++t) {
      int width = 0;
      for (size_t r = 0; r < lo.size(); ++r) {
        const int a = Tr.fc[lo[r]], b = Tr.fc[hi[r] - 1] + Tr.nch[hi[r] - 1];
        lo[r] = a;
        hi[r] = b;
        width = std::max(width, b - a);
      }
      if (width > 1 && width * tiles > kShWaves) {  // stage t opens a segment
        L.cut.push_back(t);
        const int n = Tr.stage_off[t + 1] - Tr.stage_off[t];
        lo.resize(n);
        hi.resize(n);
        for (int r = 0; r < n; ++r) {
          lo[r] = Tr.stage_off[t] + r;
          hi[r] = lo[r] + 1;
        }
      }
    }
  }
  L.cut.push_back(Tr.N);
  // the levels a workgroup keeps in LDS
  for (size_t k = 0; k + 1 < L.cut.size(); ++k)
    if (L.cut[k + 1] - L.cut[k] > kShMaxLevels) L.cut.insert(L.cut.begin() + k + 1, L.cut[k] + kShMaxLevels);
  return L;
}
template <typename S>
hipError_t sh_launch_sweeps(const Problem& P, const DevProb<S>& D, const ShPlan& L, S* Tv, const double* x0s, S* xbar,
                            S* ubar, S* q, S* d, long long vs, int Bp, hipStream_t st, ShDone done) {
  const Tree& Tr = *P.tree;
  const int groups = Bp / kShCols, segs = (int)L.cut.size() - 1;
  auto launch = [&](auto kernel, int k) {
    const int ta = L.cut[k], nsub = Tr.stage_off[ta + 1] - Tr.stage_off[ta];
    const ShSweepArgs A{L.maxch, ta, L.cut[k + 1], nsub};
    hipLaunchKernelGGL(kernel, dim3(groups * nsub), dim3(64 * kShWaves), 0, st, D, P.d_stage_off, Tv, x0s, xbar, ubar, q,
                       d, vs, A, done);
  };
  if (segs == 1) {
    launch(k_sh_sweeps<S, 3>, 0);
  } else {
    for (int k = segs - 1; k >= 0; --k) launch(k_sh_sweeps<S, 1>, k);
    for (int k = 0; k < segs; ++k) launch(k_sh_sweeps<S, 2>, k);
  }
  return hipGetLastError();
}

template <typename S>
hipError_t sh_launch_M(const Problem& P, const DevProb<S>& D, const ShVec<S>& V, const ShState* state, int B,
                       hipStream_t st) {
  const int T = std::max(P.nx, P.nu) <= 8 ? 8 : (std::max(P.nx, P.nu) <= 16 ? 16 : 32), tpb = 256 / T;
  const dim3 grid((P.tree->nl + tpb - 1) / tpb, B);
  switch (T) {
    case 8: hipLaunchKernelGGL((k_sh_M<S, 8>), grid, dim3(256), 0, st, D, V, state); break;
    case 16: hipLaunchKernelGGL((k_sh_M<S, 16>), grid, dim3(256), 0, st, D, V, state); break;
    default: hipLaunchKernelGGL((k_sh_M<S, 32>), grid, dim3(256), 0, st, D, V, state); break;
  }
  return hipGetLastError();
}

}  // namespace

template <typename S>
int shared_solve(Problem& P, int B, const double* const* x0, const spock_settings& s, void* const* vio,
                 spock_info* infos, hipStream_t st) {
  const Tree& Tr = *P.tree;
  const DevProb<S>& D = sh_dev<S>(P);
  const int nx = P.nx, nu = P.nu;
  const long long nv = P.nz + P.neta;
  const long long vs = (nv + 63) & ~63LL;
  const int Bp = (B + kShCols - 1) / kShCols * kShCols;
  const int nblk = sh_post_blocks(P);
  const int vblk = (int)std::min<long long>((nv + 511) / 512, 64);  // blocks of the vector passes per instance
  const size_t nvec = (size_t)Bp * vs;
  // device layout
  size_t off = 0;
  auto reserve = [&](size_t b) {
    const size_t o = off;
    off += (b + 255) & ~size_t(255);
    return o;
  };
  const size_t o_vec = reserve(sizeof(S) * nvec * (7 + 2 * kAAMax));
  const size_t o_qx = reserve(sizeof(S) * (size_t)Bp * Tr.nn * nx * 2);
  const size_t o_du = reserve(sizeof(S) * (size_t)Bp * Tr.nn * nu * 2);
  const size_t o_x0 = reserve(sizeof(double) * (size_t)Bp * nx);
  const size_t o_part = reserve(sizeof(double) * (size_t)Bp * nblk * kStats);
  const size_t o_dots = reserve(sizeof(double) * (size_t)B * vblk * (2 * kAAMax + 1));
  const size_t o_state = reserve(sizeof(ShState) * (size_t)B);
  // uploaded together: the callers' pointers, the root box, the count of ended instances
  const size_t o_io = reserve(sizeof(ShIO<S>) * (size_t)B);
  const size_t o_box = reserve(sizeof(double) * 2 * (size_t)nx);
  const size_t o_done = reserve(sizeof(unsigned));
  const size_t up_bytes = off - o_io;
  ShCache& C = sh_cache();
  if (C.bytes < off) {
    if (C.mem) (void)hipFree(C.mem);
    C.mem = nullptr;
    C.bytes = 0;
    if (hipMalloc(&C.mem, off) != hipSuccess) return SPOCK_ENOMEM;
    C.bytes = off;
  }
  const size_t hbytes = 256 + std::max(up_bytes, sizeof(ShState) * (size_t)B);
  if (C.host_bytes < hbytes) {
    if (C.host) (void)hipHostFree(C.host);
    C.host = nullptr;
    C.host_bytes = 0;
    if (hipHostMalloc(&C.host, hbytes, hipHostMallocCoherent | hipHostMallocMapped) != hipSuccess) return SPOCK_ENOMEM;
    C.host_bytes = hbytes;
  }
  ShMail* mail = static_cast<ShMail*>(C.host);
  ShMail* mail_d = nullptr;
  SH_TRY(hipHostGetDevicePointer(reinterpret_cast<void**>(&mail_d), mail, 0));
  std::memset(static_cast<void*>(mail), 0, sizeof(ShMail));
  char* up = static_cast<char*>(C.host) + 256;
  char* base = static_cast<char*>(C.mem);
  ShVec<S> V{};
  S* vb = reinterpret_cast<S*>(base + o_vec);
  S** roles[7] = {&V.v, &V.tv, &V.rcur, &V.dir, &V.md, &V.vt, &V.tvt};
  for (int r = 0; r < 7; ++r) *roles[r] = vb + (size_t)r * nvec;
  V.E = vb + (size_t)7 * nvec;
  V.R = V.E + (size_t)kAAMax * nvec;
  V.vs = vs;
  V.nv = nv;
  V.slot = (long long)nvec;
  S* q = reinterpret_cast<S*>(base + o_qx);
  S* xbar = q + (size_t)Bp * Tr.nn * nx;
  S* d = reinterpret_cast<S*>(base + o_du);
  S* ubar = d + (size_t)Bp * Tr.nn * nu;
  double* x0s = reinterpret_cast<double*>(base + o_x0);
  double* partials = reinterpret_cast<double*>(base + o_part);
  double* dots = reinterpret_cast<double*>(base + o_dots);
  double* rdots = dots + (size_t)B * vblk * (2 * kAAMax);
  ShState* state = reinterpret_cast<ShState*>(base + o_state);
  const ShIO<S>* io = reinterpret_cast<const ShIO<S>*>(base + o_io);
  const double* box = reinterpret_cast<const double*>(base + o_box);
  unsigned* done = reinterpret_cast<unsigned*>(base + o_done);
  // ---- inputs
  {
    std::memset(up, 0, up_bytes);
    ShIO<S>* hio = reinterpret_cast<ShIO<S>*>(up);
    for (int b = 0; b < B; ++b) hio[b] = ShIO<S>{x0[b], static_cast<S*>(vio[b])};
    double* hbox = reinterpret_cast<double*>(up + (o_box - o_io));
    std::copy(P.xlo0.begin(), P.xlo0.end(), hbox);
    std::copy(P.xhi0.begin(), P.xhi0.end(), hbox + nx);
    SH_TRY(hipMemcpyAsync(base + o_io, up, up_bytes, hipMemcpyHostToDevice, st));
  }
  const dim3 vgrid(vblk, B);
  hipLaunchKernelGGL(k_sh_load<S>, dim3(vblk, Bp), dim3(256), 0, st, V, io, B, nx, s.m, box, x0s, state, done);
  SH_TRY(hipGetLastError());
  const ShSettings S3{s.eps_abs, s.eps_rel, s.c0, s.c1, s.c2, s.beta, s.sigma, s.lambda, s.max_iters, s.max_ls, s.m,
                      s.method == SPOCK_METHOD_CP ? 1 : 0};
  const ShPlan plan = sh_plan(P);
  // ---- rounds: one evaluation of T for every instance each; the host stays
  // one round ahead of the count of ended instances
  const ShDone ended{done, (unsigned)B};
  auto wait_round = [&](unsigned long long r) -> int {
    for (unsigned n = 1;; ++n) {
      if (__atomic_load_n(&mail->round, __ATOMIC_ACQUIRE) >= r) return SPOCK_OK;
      if ((n & 4095u) == 0u) {
        const hipError_t e = hipStreamQuery(st);
        if (e == hipSuccess) return __atomic_load_n(&mail->round, __ATOMIC_ACQUIRE) >= r ? SPOCK_OK : SPOCK_EHIP;
        if (e != hipErrorNotReady) return SPOCK_EHIP;
      }
    }
  };
  for (unsigned long long r = 1;; ++r) {
    SH_TRY(sh_launch_pre<S>(P, D, V.vt, V.tvt, xbar, ubar, q, vs, Bp, st));
    SH_TRY(sh_launch_sweeps<S>(P, D, plan, V.tvt, x0s, xbar, ubar, q, d, vs, Bp, st, ended));
    SH_TRY(sh_launch_post<S>(P, D, V.vt, V.tvt, vs, partials, Bp, st));
    if (!S3.cp) hipLaunchKernelGGL(k_sh_rdot<S>, vgrid, dim3(256), 0, st, V, state, rdots);
    hipLaunchKernelGGL(k_sh_judge, dim3(B), dim3(256), 0, st, state, S3, partials, nblk, rdots, vblk, P.alpha, done);
    hipLaunchKernelGGL(k_sh_commit<S>, vgrid, dim3(256), 0, st, V, state, S3.cp, dots);
    hipLaunchKernelGGL(k_sh_plan, dim3(B), dim3(256), 0, st, state, S3, dots, vblk, done);
    hipLaunchKernelGGL(k_sh_next<S>, vgrid, dim3(256), 0, st, V, state, B, io, done, mail_d, r);
    if (!S3.cp) SH_TRY(sh_launch_M<S>(P, D, V, state, B, st));
    SH_TRY(hipGetLastError());
    if (r > 1) {
      if (int rc = wait_round(r - 1)) return rc;
      if (__atomic_load_n(&mail->done, __ATOMIC_RELAXED) >= (unsigned long long)B) break;
    }
  }
  ShState* hs = reinterpret_cast<ShState*>(up);
  SH_TRY(hipMemcpyAsync(hs, state, sizeof(ShState) * (size_t)B, hipMemcpyDeviceToHost, st));
  SH_TRY(hipStreamSynchronize(st));
  for (int b = 0; b < B; ++b) {
    const ShState& I = hs[b];
    spock_info n{};
    n.status = I.status;
    n.mapping = kTeamShared;
    n.V_nested = std::numeric_limits<double>::quiet_NaN();
    if (I.status != SPOCK_REJECTED) {
      n.iters = I.k;
      n.t_evals = I.t_evals;
      n.n_k0 = I.n_k0;
      n.n_k1 = I.n_k1;
      n.n_k2 = I.n_k2;
      n.n_km = I.n_km;
      n.n_backtracks = I.n_bt;
      n.xi0 = I.xi0;
      n.xi = I.xi;
      n.V_s0 = I.s0;
    }
    infos[b] = n;
  }
  return SPOCK_OK;
}

// ================================================================ batched adjoint
// The adjoint fixed point of section 3 (see spock_backward) for B instances
// of one problem at once: every vector holds the instances `vs` elements
// apart, the S1 part of J_T' runs the shared-tree sweeps above (zero root
// state, zero dual), J_G, L and L* run with an instance grid dimension, and
// every instance runs its own restarted GMRES; the Arnoldi steps advance in
// lockstep, an instance leaving its cycle (small residual or breakdown) keeps
// computing but its columns are not used.
namespace {

// out[o_i] = a x[x_i] + c y[y_i] + e w[w_i] on entries [0, len) of every
// instance b (operand p at p.ptr + b * p.is + p.off); y, w may be null.
template <typename S>
struct BOp {
  S* p;
  long long is, off;
};
template <typename S>
__global__ void __launch_bounds__(256) k_blin3(long long len, BOp<S> out, double a, BOp<S> x, double c, BOp<S> y,
                                               double e, BOp<S> w) {
  const size_t b = blockIdx.y;
  S* o = out.p + b * out.is + out.off;
  const S* xp = x.p + b * x.is + x.off;
  const S* yp = y.p ? y.p + b * y.is + y.off : nullptr;
  const S* wp = w.p ? w.p + b * w.is + w.off : nullptr;
  for (long long k = blockIdx.x * (long long)blockDim.x + threadIdx.x; k < len; k += (long long)gridDim.x * blockDim.x) {
    double acc = a * (double)xp[k];
    if (yp) acc += c * (double)yp[k];
    if (wp) acc += e * (double)wp[k];
    o[k] = (S)acc;
  }
}

// Per instance b: out[2 b] = max_k |x_k - y_k|, out[2 b + 1] = max_k |x_k|
// over its first n entries (one block of 1024 threads per instance).
template <typename S>
__global__ void __launch_bounds__(1024) k_bmaxdiff(long long n, const S* __restrict__ x, const S* __restrict__ y,
                                                   long long is, double* __restrict__ out) {
  const size_t b = blockIdx.x;
  const S* xb = x + b * is;
  const S* yb = y + b * is;
  double m0 = 0, m1 = 0;
  for (long long k = threadIdx.x; k < n; k += blockDim.x) {
    m0 = fmax(m0, fabs((double)xb[k] - (double)yb[k]));
    m1 = fmax(m1, fabs((double)xb[k]));
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    m0 = fmax(m0, __shfl_xor(m0, m, 64));
    m1 = fmax(m1, __shfl_xor(m1, m, 64));
  }
  __shared__ double r0[16], r1[16];
  if ((threadIdx.x & 63) == 0) {
    r0[threadIdx.x >> 6] = m0;
    r1[threadIdx.x >> 6] = m1;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double a0 = 0, a1 = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
      a0 = fmax(a0, r0[w]);
      a1 = fmax(a1, r1[w]);
    }
    out[2 * b] = a0;
    out[2 * b + 1] = a1;
  }
}

// Krylov basis of instance b at basis + b * bs (vector j at + j * vs), its
// vector x at x + b * xs. k_bdots: block (c, j, b) sums chunk c of <V_j, x>
// (j < n; <x, x> for j = n) into part[(b * m + j) * cb + c], m = gridDim.y;
// k_bdots_final (block b) adds the chunks in order into out[b * ldo + j], and
// into host (mapped pinned memory) too when given.
template <typename S>
__global__ void __launch_bounds__(256) k_bdots(long long nv, int n, const S* __restrict__ basis, long long bs,
                                               long long vs, const S* __restrict__ x, long long xs,
                                               double* __restrict__ part) {
  const int j = blockIdx.y, m = gridDim.y;
  const size_t b = blockIdx.z;
  const S* xb = x + b * xs;
  const S* v = j < n ? basis + b * bs + (size_t)j * vs : xb;
  const long long chunk = (nv + gridDim.x - 1) / gridDim.x;
  const long long e0 = (long long)blockIdx.x * chunk;
  const long long e1 = e0 + chunk < nv ? e0 + chunk : nv;
  double acc = 0;
  for (long long e = e0 + threadIdx.x; e < e1; e += 256) acc += (double)v[e] * (double)xb[e];
#pragma unroll
  for (int k = 32; k >= 1; k >>= 1) acc += __shfl_xor(acc, k, 64);
  __shared__ double red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0)
    part[((size_t)b * m + j) * gridDim.x + blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}
__global__ void __launch_bounds__(256) k_bdots_final(const double* __restrict__ part, int cb, int m,
                                                     double* __restrict__ out, int ldo, double* __restrict__ host) {
  const size_t b = blockIdx.x;
  for (int j = threadIdx.x; j < m; j += blockDim.x) {
    double acc = 0;
    for (int c = 0; c < cb; ++c) acc += part[((size_t)b * m + j) * cb + c];
    out[b * ldo + j] = acc;
    if (host) host[b * ldo + j] = acc;
  }
}
// x_b += sgn sum_{j < n} c_b[j] V_j (c_b = c + b * ldc, device); with norm,
// then scaled by 1 / sqrt(c_b[n] - sum_j c_b[j]^2) (0 if not positive)
template <typename S>
__global__ void __launch_bounds__(256) k_bcomb(long long nv, int n, const S* __restrict__ basis, long long bs,
                                               long long vs, const double* __restrict__ c, int ldc, double sgn,
                                               int norm, S* x, long long xs) {
  const size_t b = blockIdx.y;
  const double* cb = c + b * ldc;
  const S* Vb = basis + b * bs;
  S* xb = x + b * xs;
  double scale = 1.0;
  if (norm) {
    double h2 = cb[n];
    for (int j = 0; j < n; ++j) h2 -= cb[j] * cb[j];
    scale = h2 > 0.0 ? 1.0 / sqrt(h2) : 0.0;
  }
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < nv; e += (long long)gridDim.x * blockDim.x) {
    double acc = (double)xb[e];
    for (int j = 0; j < n; ++j) acc += sgn * cb[j] * (double)Vb[(size_t)j * vs + e];
    xb[e] = (S)(acc * scale);
  }
}

}  // namespace

template <typename S>
int shared_backward(Problem& P, int B, const void* const* vstar, const double* const* x0, double gV,
                    const double* const* gu0, double* const* gx0, double* const* gq, double* const* gqN,
                    const spock_settings& s, spock_info* infos, hipStream_t st) {
  const Tree& Tr = *P.tree;
  const DevProb<S>& D = sh_dev<S>(P);
  const int nx = P.nx, nu = P.nu;
  const long long nz = P.nz, ne = P.neta, nv = nz + ne;
  const long long vs = (nv + 63) & ~63LL;
  const int Bp = (B + kShCols - 1) / kShCols * kShCols;
  const double al = P.alpha;
  constexpr int kMax = 120;  // Krylov vectors per cycle at most
  int R = sizeof(S) * (size_t)(kMax + 1) * (size_t)vs * (size_t)Bp <= (size_t(2) << 30) ? kMax : 30;
  if (const char* env = std::getenv("SPOCK_ADJ_RESTART")) R = std::max(2, std::min(kMax, std::atoi(env)));
  const long long bs = (long long)(R + 1) * vs;  // basis stride between instances
  const int cb = std::max(1, std::min(64, (int)((nv + 8191) / 8192)));
  const int ldc = kMax + 2;
  // ---- device memory: 13 batch vectors, the bases, sweep buffers, x0s,
  // coefficients and partial sums
  enum { kV, kTv, kDz, kLdz, kB, kG, kW, kAw, kLb, kCz, kLa, kTz, kIn, kNVec };
  const size_t nvec = (size_t)Bp * vs;
  size_t off = 0;
  auto reserve = [&](size_t bytes) {
    const size_t o = off;
    off += (bytes + 255) & ~size_t(255);
    return o;
  };
  const size_t o_vec = reserve(sizeof(S) * nvec * kNVec);
  const size_t o_bas = reserve(sizeof(S) * (size_t)Bp * bs);
  const size_t o_qx = reserve(sizeof(S) * (size_t)Bp * Tr.nn * nx * 2);
  const size_t o_du = reserve(sizeof(S) * (size_t)Bp * Tr.nn * nu * 2);
  const size_t o_x0 = reserve(sizeof(double) * (size_t)Bp * nx * 2);
  const size_t o_c = reserve(sizeof(double) * (size_t)Bp * ldc * 3);
  const size_t o_part = reserve(sizeof(double) * (size_t)Bp * (kMax + 2) * cb);
  const size_t o_md = reserve(sizeof(double) * (size_t)Bp * 2);
  const size_t o_mu = reserve(sizeof(S) * (size_t)B * Tr.nn * nx);
  const size_t o_tab = reserve(sizeof(AdjPtrs<S>) * (size_t)B);
  void* mem = nullptr;
  if (hipMalloc(&mem, off) != hipSuccess) return SPOCK_ENOMEM;
  struct Guard {
    void* m;
    ~Guard() { (void)hipFree(m); }
  } guard{mem};
  char* base = static_cast<char*>(mem);
  // padding instances stay at zero; a basis vector is written (by every
  // instance) before anything reads it
  SH_TRY(hipMemsetAsync(base, 0, o_bas, st));
  SH_TRY(hipMemsetAsync(base + o_qx, 0, off - o_qx, st));
  S* vec[kNVec];
  for (int r = 0; r < kNVec; ++r) vec[r] = reinterpret_cast<S*>(base + o_vec) + (size_t)r * nvec;
  S* basis = reinterpret_cast<S*>(base + o_bas);
  S* q = reinterpret_cast<S*>(base + o_qx);
  S* xbar = q + (size_t)Bp * Tr.nn * nx;
  S* d = reinterpret_cast<S*>(base + o_du);
  S* ubar = d + (size_t)Bp * Tr.nn * nu;
  double* x0s = reinterpret_cast<double*>(base + o_x0);
  double* x0zero = x0s + (size_t)Bp * nx;
  double* cdev = reinterpret_cast<double*>(base + o_c);  // [Bp][ldc] x 3: pass 1, pass 2, mix
  double* c1 = cdev;
  double* c2 = cdev + (size_t)Bp * ldc;
  double* cm = cdev + 2 * (size_t)Bp * ldc;
  double* part = reinterpret_cast<double*>(base + o_part);
  double* md = reinterpret_cast<double*>(base + o_md);
  S* mu = reinterpret_cast<S*>(base + o_mu);
  AdjPtrs<S>* tab_d = reinterpret_cast<AdjPtrs<S>*>(base + o_tab);
  const int vb = (int)std::min<long long>((nv + 255) / 256, 64);
  auto op = [&](int r, long long o = 0) { return BOp<S>{vec[r], vs, o}; };
  auto lin3 = [&](long long len, BOp<S> o, double a, BOp<S> x, double c = 0, BOp<S> y = BOp<S>{nullptr, 0, 0},
                  double e = 0, BOp<S> w = BOp<S>{nullptr, 0, 0}) -> int {
    hipLaunchKernelGGL(k_blin3<S>, dim3(vb, Bp), dim3(256), 0, st, len, o, a, x, c, y, e, w);
    SH_TRY(hipGetLastError());
    return SPOCK_OK;
  };
  // ---- inputs: v* and x0 of every instance, the cotangents and w = g
  std::vector<AdjPtrs<S>> tab(B);
  for (int b = 0; b < B; ++b)
    tab[b] = AdjPtrs<S>{static_cast<const S*>(vstar[b]), x0[b], gu0 ? gu0[b] : nullptr,
                        gx0[b], gq ? gq[b] : nullptr, gqN ? gqN[b] : nullptr};
  SH_TRY(hipMemcpyAsync(tab_d, tab.data(), sizeof(AdjPtrs<S>) * B, hipMemcpyHostToDevice, st));
  SH_TRY(launch_adj_load<S>(P, gV, tab_d, vs, B, vec[kV], x0s, vec[kG], vec[kW], st));
  // (every sweep runs: any word below the largest)
  const ShDone never{reinterpret_cast<const unsigned*>(P.d_stage_off), ~0u};
  // prox_f of the instances: pre-pass, then the sweeps
  const ShPlan plan = sh_plan(P);
  auto prox = [&](S* in, S* out, const double* xs0) -> int {
    SH_TRY(sh_launch_pre<S>(P, D, in, out, xbar, ubar, q, vs, Bp, st));
    SH_TRY(sh_launch_sweeps<S>(P, D, plan, out, xs0, xbar, ubar, q, d, vs, Bp, st, never));
    return SPOCK_OK;
  };
  // pre-prox point of the dual update at v*: b* = eta* + alpha L (2 z+ - z*)
  if (int r = prox(vec[kV], vec[kTv], x0s)) return r;
  if (int r = lin3(nz, op(kDz), 2.0, op(kTv), -1.0, op(kV))) return r;
  SH_TRY(launch_L_batch<S>(P, vec[kDz], vec[kLdz], vs, Bp, st));
  if (int r = lin3(ne, op(kB), 1.0, op(kV, nz), al, op(kLdz))) return r;
  // one application of the transposed operator to w (instances ws apart): lb, tz, cz, la
  const bool fused = plan.maxch <= kAdjMaxCh;
  auto partial = [&](const S* w, long long ws) -> int {
    if (fused) {
      SH_TRY(launch_adj_front<S>(P, vec[kB], w, ws, vec[kLb], vec[kTz], vec[kCz], vec[kLa], xbar, ubar, q, vs, Bp,
                                 true, st));
      SH_TRY(sh_launch_sweeps<S>(P, D, plan, vec[kLa], x0zero, xbar, ubar, q, d, vs, Bp, st, never));
      return SPOCK_OK;
    }
    if (w != vec[kIn])
      SH_TRY(hipMemcpy2DAsync(vec[kIn], sizeof(S) * vs, w, sizeof(S) * ws, sizeof(S) * nv, Bp, hipMemcpyDeviceToDevice, st));
    SH_TRY(launch_jg_batch<S>(P, vec[kB], vec[kIn] + nz, vec[kLb], vs, Bp, st));  // lambda_b = J_G w_eta
    SH_TRY(launch_Lt_batch<S>(P, vec[kLb], vec[kTz], vs, Bp, st));                // L* lambda_b
    if (int r = lin3(nz, op(kCz), 1.0, op(kIn), 2.0 * al, op(kTz))) return r;     // w_z + 2 alpha L* lambda_b
    if (int r = prox(vec[kCz], vec[kLa], x0zero)) return r;                       // J_f c (zero dual part)
    if (int r = lin3(1, op(kLa), 1.0, op(kCz))) return r;                         // identity on s^0
    return SPOCK_OK;
  };
  // out = a w + sg J_T(v*)' w + cg g after partial(w)
  auto back = [&](double a, const S* w, long long ws, double sg, double cg, S* out, long long os) -> int {
    SH_TRY(launch_adj_back<S>(P, a, w, ws, sg, vec[kLa], vec[kTz], vec[kLb], cg, vec[kG], out, os, vs, Bp, st));
    return SPOCK_OK;
  };
  auto bdots = [&](int n, const S* x, long long xs, bool xx, double* out, double* hout = nullptr) -> int {
    const int m = n + (xx ? 1 : 0);
    hipLaunchKernelGGL(k_bdots<S>, dim3(cb, m, Bp), dim3(256), 0, st, nv, n, basis, bs, vs, x, xs, part);
    hipLaunchKernelGGL(k_bdots_final, dim3(Bp), dim3(256), 0, st, part, cb, m, out, ldc, hout);
    SH_TRY(hipGetLastError());
    return SPOCK_OK;
  };
  auto bcomb = [&](int n, const double* c, double sgn, bool norm, S* x, long long xs) -> int {
    hipLaunchKernelGGL(k_bcomb<S>, dim3(vb, Bp), dim3(256), 0, st, nv, n, basis, bs, vs, c, ldc, sgn, norm ? 1 : 0, x,
                       xs);
    SH_TRY(hipGetLastError());
    return SPOCK_OK;
  };
  auto V = [&](int j) { return basis + (size_t)j * vs; };  // vector j of instance 0 (instances bs apart)
  // ---- restarted GMRES per instance, Arnoldi steps in lockstep
  const double tol = std::max(s.eps_abs, 1e-15);
  std::vector<int> kk(B, 0), state(B, 0);  // state: 0 running, 1 converged, 2 numerical, 3 max_iters
  std::vector<double> diff(B, 0.0);
  std::vector<double> hmd((size_t)Bp * 2), hc1((size_t)Bp * ldc), hcm((size_t)Bp * ldc);
  // the Gram-Schmidt coefficients on the host: [2 slots][2 passes][Bp][ldc]
  double* hp = nullptr;
  if (hipHostMalloc(reinterpret_cast<void**>(&hp), sizeof(double) * 4 * (size_t)Bp * ldc,
                    hipHostMallocCoherent | hipHostMallocMapped) != hipSuccess)
    return SPOCK_ENOMEM;
  hipEvent_t evs[2] = {nullptr, nullptr};
  struct PipeGuard {
    double* hp;
    hipEvent_t* ev;
    hipStream_t st;
    ~PipeGuard() {
      (void)hipStreamSynchronize(st);  // an early return: queued kernels write hp
      for (int e = 0; e < 2; ++e)
        if (ev[e]) (void)hipEventDestroy(ev[e]);
      (void)hipHostFree(hp);
    }
  } pguard{hp, evs, st};
  for (int e = 0; e < 2; ++e) SH_TRY(hipEventCreateWithFlags(&evs[e], hipEventDisableTiming));
  double* hp_dev = nullptr;
  SH_TRY(hipHostGetDevicePointer(reinterpret_cast<void**>(&hp_dev), hp, 0));
  auto hslot = [&](int j, int pass) { return hp + ((size_t)(j & 1) * 2 + pass) * (size_t)Bp * ldc; };
  auto hdev = [&](int j, int pass) { return hp_dev + ((size_t)(j & 1) * 2 + pass) * (size_t)Bp * ldc; };
  std::vector<double> Hm((size_t)B * (kMax + 1) * kMax), cs((size_t)B * kMax), sn((size_t)B * kMax),
      gvv((size_t)B * (kMax + 1));
  std::vector<int> jn(B), incyc(B);
  auto running = [&]() {
    for (int b = 0; b < B; ++b)
      if (state[b] == 0) return true;
    return false;
  };
  while (running()) {
    // true residual of every instance at w
    if (int r = partial(vec[kW], vs)) return r;
    if (int r = back(0.0, vec[kW], vs, 1.0, 1.0, vec[kAw], vs)) return r;
    hipLaunchKernelGGL(k_bmaxdiff<S>, dim3(Bp), dim3(1024), 0, st, nv, vec[kW], vec[kAw], vs, md);
    SH_TRY(hipGetLastError());
    SH_TRY(hipMemcpyAsync(hmd.data(), md, sizeof(double) * 2 * Bp, hipMemcpyDeviceToHost, st));
    SH_TRY(hipStreamSynchronize(st));
    for (int b = 0; b < B; ++b) {
      if (state[b] != 0) continue;
      ++kk[b];
      diff[b] = hmd[2 * b];
      if (!std::isfinite(diff[b])) state[b] = 2;
      else if (diff[b] <= tol * std::max(1.0, hmd[2 * b + 1])) state[b] = 1;
      else if (kk[b] >= s.max_iters) state[b] = 3;
    }
    if (!running()) break;
    // V_0 = (A(w) - w) / |.| for every instance
    if (int r = lin3(nv, BOp<S>{basis, bs, 0}, 1.0, op(kAw), -1.0, op(kW))) return r;
    if (int r = bdots(0, V(0), bs, true, c1)) return r;
    SH_TRY(hipMemcpyAsync(hc1.data(), c1, sizeof(double) * Bp * ldc, hipMemcpyDeviceToHost, st));
    SH_TRY(hipStreamSynchronize(st));
    if (int r = bcomb(0, c1, 1.0, true, V(0), bs)) return r;
    std::fill(Hm.begin(), Hm.end(), 0.0);
    for (int b = 0; b < B; ++b) {
      const double beta = std::sqrt(std::max(hc1[(size_t)b * ldc], 0.0));
      gvv[(size_t)b * (kMax + 1)] = beta;
      jn[b] = 0;
      incyc[b] = state[b] == 0 && beta > 0.0 && std::isfinite(beta);
      if (state[b] == 0 && !(beta > 0.0)) state[b] = std::isfinite(beta) ? 1 : 2;
    }
    auto any_in = [&]() {
      for (int b = 0; b < B; ++b)
        if (incyc[b]) return true;
      return false;
    };
    // Arnoldi steps are pipelined as in the one-instance form: the passes take
    // their coefficients from device memory, the reductions also write them to
    // mapped pinned memory, and the host reduces column j of every instance's
    // Hessenberg matrix while step j + 1 runs (two slots, alternating). No step
    // starts that every instance's cap on applications rules out.
    auto column = [&](int j) -> int {
      SH_TRY(hipEventSynchronize(evs[j & 1]));
      for (int b = 0; b < B; ++b) {
        if (!incyc[b]) continue;
        ++kk[b];
        double* Hb = Hm.data() + (size_t)b * (kMax + 1) * kMax;
        auto H = [&](int i, int jj) -> double& { return Hb[(size_t)i * kMax + jj]; };
        double* csb = cs.data() + (size_t)b * kMax;
        double* snb = sn.data() + (size_t)b * kMax;
        double* gv = gvv.data() + (size_t)b * (kMax + 1);
        const double* h1 = hslot(j, 0) + (size_t)b * ldc;
        const double* h2 = hslot(j, 1) + (size_t)b * ldc;
        double hn = h2[j + 1];
        for (int i = 0; i <= j; ++i) {
          H(i, j) = h1[i] + h2[i];
          hn -= h2[i] * h2[i];
        }
        hn = std::sqrt(std::max(hn, 0.0));
        H(j + 1, j) = hn;
        for (int i = 0; i < j; ++i) {
          const double xv = H(i, j), yv = H(i + 1, j);
          H(i, j) = csb[i] * xv + snb[i] * yv;
          H(i + 1, j) = -snb[i] * xv + csb[i] * yv;
        }
        const double rr = std::hypot(H(j, j), H(j + 1, j));
        csb[j] = rr > 0.0 ? H(j, j) / rr : 1.0;
        snb[j] = rr > 0.0 ? H(j + 1, j) / rr : 0.0;
        H(j, j) = rr;
        H(j + 1, j) = 0.0;
        gv[j + 1] = -snb[j] * gv[j];
        gv[j] = csb[j] * gv[j];
        jn[b] = j + 1;
        const double thr = tol * std::max(1.0, hmd[2 * b + 1]);
        if (!std::isfinite(gv[j + 1]) || std::fabs(gv[j + 1]) <= 0.5 * thr || !(hn > 0.0) || kk[b] >= s.max_iters)
          incyc[b] = 0;
      }
      return SPOCK_OK;
    };
    int steps = 0;  // Arnoldi steps of the cycle at most
    for (int b = 0; b < B; ++b)
      if (incyc[b]) steps = std::max(steps, std::min(R, s.max_iters - kk[b]));
    int launched = 0;
    for (int j = 0; j < steps && any_in(); ++j) {
      if (int r = partial(V(j), bs)) return r;
      // V_{j+1} = V_j - J_T' V_j, two Gram-Schmidt passes, normalisation
      if (int r = back(1.0, V(j), bs, -1.0, 0.0, V(j + 1), bs)) return r;
      if (int r = bdots(j + 1, V(j + 1), bs, false, c1, hdev(j, 0))) return r;
      if (int r = bcomb(j + 1, c1, -1.0, false, V(j + 1), bs)) return r;
      if (int r = bdots(j + 1, V(j + 1), bs, true, c2, hdev(j, 1))) return r;
      if (int r = bcomb(j + 1, c2, -1.0, true, V(j + 1), bs)) return r;
      SH_TRY(hipEventRecord(evs[j & 1], st));
      launched = j + 1;
      if (j > 0)
        if (int r = column(j - 1)) return r;
    }
    if (launched > 0)
      if (int r = column(launched - 1)) return r;
    // w += V y per instance (H y = g, upper triangular; zero for the others)
    std::fill(hcm.begin(), hcm.end(), 0.0);
    int nmax = 0;
    for (int b = 0; b < B; ++b) {
      if (state[b] != 0 || jn[b] == 0) continue;
      const double* Hb = Hm.data() + (size_t)b * (kMax + 1) * kMax;
      const double* gv = gvv.data() + (size_t)b * (kMax + 1);
      double* y = hcm.data() + (size_t)b * ldc;
      for (int i = jn[b] - 1; i >= 0; --i) {
        double t = gv[i];
        for (int l = i + 1; l < jn[b]; ++l) t -= Hb[(size_t)i * kMax + l] * y[l];
        y[i] = Hb[(size_t)i * kMax + i] != 0.0 ? t / Hb[(size_t)i * kMax + i] : 0.0;
      }
      nmax = std::max(nmax, jn[b]);
    }
    SH_TRY(hipMemcpyAsync(cm, hcm.data(), sizeof(double) * Bp * ldc, hipMemcpyHostToDevice, st));
    if (int r = bcomb(nmax, cm, 1.0, false, vec[kW], vs)) return r;
    SH_TRY(hipStreamSynchronize(st));  // hcm is reused
  }
  // gradients from the converged adjoints
  if (int r = partial(vec[kW], vs)) return r;
  SH_TRY(launch_phiT<S>(P, vec[kCz], vs, mu, (long long)Tr.nn * nx, B, tab_d, st));
  if (gq || gqN) SH_TRY(launch_grad_q<S>(P, vec[kV], vec[kLa], vec[kLb], vs, B, tab_d, st));
  for (int b = 0; b < B; ++b) {
    spock_info loc{};
    loc.V_nested = std::numeric_limits<double>::quiet_NaN();
    loc.status = state[b] == 1 ? SPOCK_CONVERGED : (state[b] == 2 ? SPOCK_NUMERICAL : SPOCK_MAXITER);
    loc.iters = kk[b];
    loc.t_evals = kk[b];
    loc.xi = diff[b];
    loc.mapping = kTeamShared;
    infos[b] = loc;
  }
  SH_TRY(hipStreamSynchronize(st));
  return SPOCK_OK;
}

template int shared_backward<double>(Problem&, int, const void* const*, const double* const*, double,
                                     const double* const*, double* const*, double* const*, double* const*,
                                     const spock_settings&, spock_info*, hipStream_t);
template int shared_backward<float>(Problem&, int, const void* const*, const double* const*, double,
                                    const double* const*, double* const*, double* const*, double* const*,
                                    const spock_settings&, spock_info*, hipStream_t);

template int shared_solve<double>(Problem&, int, const double* const*, const spock_settings&, void* const*,
                                  spock_info*, hipStream_t);
template int shared_solve<float>(Problem&, int, const double* const*, const spock_settings&, void* const*,
                                 spock_info*, hipStream_t);

}  // namespace spk
