// Batched block engine: one workgroup per instance runs the whole SPOCK
// iteration (Alg. 3 with Anderson directions, section 6) on its own tree
// without returning to the host. Trees of different shapes and sizes share
// one launch.
//
// The evaluation of T (section 3) is arranged so that only one short mat-vec
// per stage stays on the recursion of each Alg. 2 sweep; everything else runs
// over the whole tree at once between workgroup barriers:
//   pre    xbar, ubar = (x, u) - alpha L* eta and the S2 projection, a team of
//          T lanes per family; then q = P1 ubar - xbar (-xbar at a leaf)
//   chain  stage N-1 .. 1:  q^i += sum_c At^c q^c       (one mat-vec)
//   mid    d^i = R~^{-1} ubar + sum_c Bt^c q^c, then x^c = B^c d^i (x^0 the
//          root state)
//   chain  stage 0 .. N-1:  x^c += Abar^c x^i           (one mat-vec)
//   post   u^i = K x^i + d^i, then the dual update and the residual statistics
//          (flat_family, flat_leaf), a team per family or leaf
// (the regrouped recursion: At, Bt, P1 formed in FP64 at upload). The mat-vecs
// run one thread per output over all nodes, so no lane idles on the teams'
// remainder; q and x share one buffer (x^c takes q^c's place once d^{anc c} is
// formed); it, ubar, d and the tree's index arrays sit in LDS when the largest
// tree of the batch fits, and the first matrix rows of the next stage are
// loaded into registers before the barrier that ends a stage.
//
// What bounds it: for one instance the latency of the loads from memory (the
// iterates of a batch exceed the L2: about 4000 cycles a dependent level with
// every CU at work, five levels a family in the pre- and post-pass) and of the
// stages, about 0.26 ms per iteration of a 511-node tree (n_x 10, n_u 5, FP32);
// 1024 threads at 128 registers give four wavefronts per SIMD to cover it. For
// many, the vector passes' traffic too (31 GB/s per CU in the push, 8 TB/s in
// all). 128 registers do not hold the iteration's state in either precision:
// FP32 (16 lanes, form in LDS) spills 148 vector and 477 scalar registers (592
// bytes of scratch a lane), FP64 (32 lanes) 180 and 382 (704 bytes). Six FP32
// SPOCK iterations of 512 trees (5 to 511 nodes): 10.8 -> 1.93 ms; eight FP64
// iterations of 60 trees (n_x 13, n_u 7): 11.4 -> 2.70 ms, against 256 threads
// with a team per family, two mat-vec phases a stage and flat accesses. Of
// that, largest trees first: 2.63 -> 2.0 ms; accesses known to be global with
// 32-bit offsets: 3.8 -> 2.63 ms.
#include "device_common.h"

#include <algorithm>
#include <type_traits>

namespace spk {

namespace {

constexpr int kBT = 1024;              // threads per instance
constexpr int kBW = kBT / 64;          // wavefronts per instance
constexpr int kBPool = 10 + 2 * kAAMax;  // vectors of the workspace
constexpr int kBLds = 152 * 1024;      // dynamic LDS a workgroup may take (160 KiB per CU)

// Workgroup barrier that orders LDS accesses only (global loads stay in flight).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Fixed-order sums of K per-thread values over the workgroup (the last two
// as maxima when MAX): wavefront butterflies, then the wavefronts in order;
// every thread gets the results. red holds K kBW doubles.
template <int K, bool MAX>
__device__ __forceinline__ void blk_reduce(double (&v)[K], double* red) {
  constexpr int ks = MAX ? K - 2 : K;
#pragma unroll
  for (int j = 0; j < K; ++j) v[j] = j < ks ? team_sum<64>(v[j]) : wave_max(v[j]);
  __syncthreads();  // earlier readers of red are done
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int j = 0; j < K; ++j) red[j * kBW + (threadIdx.x >> 6)] = v[j];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < K; ++j) {
    double a = red[j * kBW];
    for (int w = 1; w < kBW; ++w) a = j < ks ? a + red[j * kBW + w] : fmax(a, red[j * kBW + w]);
    v[j] = a;
  }
}

struct BStats {
  double xip = 0, xid = 0, om2 = 0;
  __device__ double xi() const { return fmax(xip, xid); }
  __device__ double omega() const { return sqrt(fmax(om2, 0.0)); }
  __device__ bool ok() const { return isfinite(xip) && isfinite(xid) && isfinite(om2); }
};

// The dynamic LDS of the form in LDS: q/x [nn][nx], ubar and d [nl][nu], the
// index arrays fc [nl], nch [nl], anc [nn] and the stage offsets [N + 2] of
// the largest tree.
struct BLds {
  long long u, d, fc, nch, anc, so, total;
};
BLds blk_lds(long long elem, const BatchShape& sh) {
  BLds L;
  auto up = [](long long b) { return (b + 15) & ~15LL; };
  L.u = up(elem * sh.nn * sh.nx);
  L.d = L.u + up(elem * sh.nl * sh.nu);
  L.fc = L.d + up(elem * sh.nl * sh.nu);
  L.nch = L.fc + up(sh.nl * 4LL);
  L.anc = L.nch + up(sh.nl * 4LL);
  L.so = L.anc + up(sh.nn * 4LL);
  L.total = L.so + up((sh.N + 2LL) * 4);
  return L;
}

// A pointer read from memory is generic to the compiler (flat accesses, which
// also wait on the LDS counter); the descriptors' pointers are all global.
template <typename U>
__device__ __forceinline__ U* as_global(U* p) {
  auto g = (__attribute__((address_space(1))) U*)p;
  asm("" : "+s"(g));  // keeps the cast: a cast and its inverse cancel
  return (U*)g;
}
template <typename S>
__device__ __forceinline__ DevProb<S> global_prob(const DevProb<S>& Q) {
  DevProb<S> P = Q;
  P.fc = as_global(Q.fc);
  P.nch = as_global(Q.nch);
  P.anc = as_global(Q.anc);
  P.p = as_global(Q.p);
  P.a = as_global(Q.a);
  P.sq = as_global(Q.sq);
  P.sr = as_global(Q.sr);
  P.sqN = as_global(Q.sqN);
  P.xlo = as_global(Q.xlo);
  P.xhi = as_global(Q.xhi);
  P.ulo = as_global(Q.ulo);
  P.uhi = as_global(Q.uhi);
  P.AbC = as_global(Q.AbC);
  P.BC = as_global(Q.BC);
  P.KC = as_global(Q.KC);
  P.Rinv = as_global(Q.Rinv);
  P.AtR = as_global(Q.AtR);
  P.BtR = as_global(Q.BtR);
  P.P1C = as_global(Q.P1C);
  return P;
}

// 16-byte vector of S (the workspace vectors are 256-byte aligned)
template <typename S>
struct alignas(16) Vec16 {
  S e[16 / sizeof(S)];
};

// The Gram solve of a push by one thread, out of line: its registers are not
// the iteration's.
template <int MO>
__device__ __noinline__ void blk_gram_solve(double* G, const double* dots_in, const AAPush* ap, double* gamma,
                                            AARingDev* ring) {
  const AAPush a = *ap;
  double dots[8], Gold[16];
#pragma unroll
  for (int j = 0; j < 8; ++j) dots[j] = j < 2 * MO + 2 ? dots_in[j] : 0.0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      Gold[i * 4 + j] = (i < MO && j < MO) ? G[a.order_old[i] * a.m + a.order_old[j]] : 0.0;
  aa_solve_dev<MO>(G, dots, Gold, a, gamma, ring);
}

template <typename S, int T, int SL, bool LQ>
struct BlockSolver {
  static constexpr int kTeams = kBT / T;
  // matrix rows of the next stage held in registers
  static constexpr int kPre = sizeof(S) == 8 ? 16 : 24;
  static constexpr int W = 16 / (int)sizeof(S);
  // offsets in the problem's and the iterate's arrays: 32 bits suffice for a
  // tree whose states fit the LDS (its arrays stay far below 4 GiB)
  using IX = std::conditional_t<LQ, unsigned, long long>;

  // copies: through a reference every access would load the descriptor again
  DevProb<S> P;  // the index arrays moved to LDS where they fit
  const BatchSettings s;
  const int* stage_off;
  const double* x0;
  S* vio;
  S* work;
  long long nv;
  double* red;  // [8 kBW]
  S* qx;        // [nn][nx] q, then x
  S* uu;        // [nl][nu] ubar
  S* dd;        // [nl][nu] d, then u+
  const int* so;
  int lane, team;
  // node and component of this thread's first element of a pass over [.][nx]
  // (ex, ox) and [.][nu] (eu, ou), and what kBT elements further adds to them
  int ex, ox, eu, ou, sx, rx, su, ru;
  long long nvs;  // stride of the workspace vectors

  __device__ BlockSolver(const BatchInst<S>& inst, const BatchSettings& st, unsigned char* smem, const BLds& L, double* r)
      : P(global_prob(inst.P)), s(st), stage_off(as_global(inst.stage_off)), x0(as_global(inst.x0)), vio(as_global(inst.vio)), work(as_global(inst.work)), nv(inst.nv), red(r) {
    lane = threadIdx.x % T;
    team = threadIdx.x / T;
    ex = (int)(threadIdx.x / (unsigned)P.nx);
    ox = (int)threadIdx.x - ex * P.nx;
    eu = (int)(threadIdx.x / (unsigned)P.nu);
    ou = (int)threadIdx.x - eu * P.nu;
    sx = kBT / P.nx;
    rx = kBT - sx * P.nx;
    su = kBT / P.nu;
    ru = kBT - su * P.nu;
    nvs = (nv + 63) & ~63LL;
    if constexpr (LQ) {
      qx = reinterpret_cast<S*>(smem);
      uu = reinterpret_cast<S*>(smem + L.u);
      dd = reinterpret_cast<S*>(smem + L.d);
      int* f = reinterpret_cast<int*>(smem + L.fc);
      int* c = reinterpret_cast<int*>(smem + L.nch);
      int* a = reinterpret_cast<int*>(smem + L.anc);
      int* o = reinterpret_cast<int*>(smem + L.so);
      for (int k = threadIdx.x; k < P.nn; k += kBT) {
        a[k] = P.anc[k];
        if (k < P.nl) {
          f[k] = P.fc[k];
          c[k] = P.nch[k];
        }
      }
      for (int k = threadIdx.x; k < P.N + 2; k += kBT) o[k] = stage_off[k];
      P.fc = f;
      P.nch = c;
      P.anc = a;
      so = o;
    } else {
      qx = work + (size_t)kBPool * nvs;
      uu = qx + (size_t)P.nn * P.nx;
      dd = uu + (size_t)P.nl * P.nu;
      so = stage_off;
    }
    __syncthreads();
  }
  __device__ S* pool(int k) const { return work + (size_t)k * nvs; }
  // barrier between the stages of a chain
  __device__ void stage_barrier() const {
    if constexpr (LQ) lds_barrier();
    else __syncthreads();
  }

  // Whether n is the same in every active lane; then nn is it, in a scalar
  // register (rows of a stage, as a rule), else the largest
  __device__ static bool same_rows(int n, int& nn) {
    nn = __builtin_amdgcn_readfirstlane(n);
    return __all(n == nn);
  }
  // sum_{r0 <= r < n} M[off + r ld] v[r]; n and ld uniform: the row advance is
  // scalar arithmetic, one load and one multiply-add per row on the lane
  __device__ static S dot_u(const S* M, IX off, int r0, int n, int ld, const S* v) {
    S a0 = 0, a1 = 0;
    int r = r0;
    for (; r + 4 <= n; r += 4) {
      S m[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) m[k] = at<S, IX>(M + (size_t)(r + k) * ld, off);
#pragma unroll
      for (int k = 0; k < 4; k += 2) {
        a0 += m[k] * v[r + k];
        a1 += m[k + 1] * v[r + k + 1];
      }
    }
    for (; r < n; ++r) a0 += at<S, IX>(M + (size_t)r * ld, off) * v[r];
    return a0 + a1;
  }
  // the same with n of the lane
  __device__ static S dot_n(const S* M, IX off, int n, int ld, const S* v) {
    int nu_;
    if (same_rows(n, nu_)) return dot_u(M, off, 0, nu_, ld, v);
    S a0 = 0;
    for (int r = 0; r < n; ++r) a0 += at<S, IX>(M, off + (IX)r * ld) * v[r];
    return a0;
  }
  // The first kPre rows into registers (n uniform), and the sum that uses them
  __device__ static void load_rows(S (&m)[kPre], const S* M, IX off, int n, int ld) {
#pragma unroll
    for (int r = 0; r < kPre; r += 2)
      if (r < n) {
        m[r] = at<S, IX>(M + (size_t)r * ld, off);
        m[r + 1] = at<S, IX>(M + (size_t)(r + 1 < n ? r + 1 : r) * ld, off);
      }
  }
  __device__ static S dot_rows(const S (&m)[kPre], const S* M, IX off, int n, int ld, const S* v) {
    S a0 = 0, a1 = 0;
#pragma unroll
    for (int r = 0; r < kPre; r += 2) {
      if (r + 1 < n) {
        a0 += m[r] * v[r];
        a1 += m[r + 1] * v[r + 1];
      } else if (r < n) {
        a0 += m[r] * v[r];
      }
    }
    S acc = a0 + a1;
    if (n > kPre) acc += dot_u(M, off, kPre, n, ld, v);
    return acc;
  }

  // f(node, component, element) over nodes first .. last - 1 with nx (or nu)
  // components each, a thread per element
  template <typename F>
  __device__ void each_x(int first, int last, F&& f) const {
    for (int i = first + ex, o = ox; i < last; i += sx, o += rx) {
      if (o >= P.nx) {
        o -= P.nx;
        if (++i >= last) break;
      }
      f(i, o, (IX)i * P.nx + o);
    }
  }
  template <typename F>
  __device__ void each_u(int first, int last, F&& f) const {
    for (int i = first + eu, o = ou; i < last; i += su, o += ru) {
      if (o >= P.nu) {
        o -= P.nu;
        if (++i >= last) break;
      }
      f(i, o, (IX)i * P.nu + o);
    }
  }

  // Tv = T(v) and the residual statistics of v - T(v)
  __device__ BStats Teval(const S* v, S* Tv) const {
    const S* z = v;
    const S* eta = v + P.nz;
    S* zout = Tv;
    S* eout = Tv + P.nz;
    const Off<S, IX> O(P);
    const int nx = P.nx, nu = P.nu, N = P.N;
    // ---- pre
    for (int i = team; i < P.nl; i += kTeams) {
      S b[SL];
      flat_pre_family<S, T, SL, IX>(P, O, z, eta, zout, i, P.fc[i], P.nch[i], lane, b);
#pragma unroll
      for (int k = 0; k < SL; ++k) {
        const int o = lane + T * k;
        if (o < nx) qx[(size_t)i * nx + o] = -b[k];
        else if (o < nx + nu) uu[(size_t)i * nu + (o - nx)] = b[k];
      }
    }
    each_x(P.nl, P.nn, [&](int j, int o, IX e) {
      const IX e3 = O.e3(j) + o;
      qx[e] = P.alpha * (at<S, IX>(eta, e3) + at<S, IX>(P.sqN, e) * at<S, IX>(eta, e3 + nx)) - at<S, IX>(z, 1 + e);
    });
    __syncthreads();
    each_x(1, P.nl, [&](int i, int o, IX e) {
      qx[e] += dot_u(P.P1C, (IX)i * (nu * nx) + o, 0, nu, nx, uu + (size_t)i * nu);
    });
    // ---- backward chain; the first rows of the next two stages in registers
    // (a stage is shorter than a load from memory)
    S m0[kPre], m1[kPre];
    int r0 = 0, r1 = 0;  // rows of a stage's first elements, when held
    auto fetch_b = [&](int t, S(&m)[kPre], int& rows) {
      rows = 0;
      if (t < 1) return;
      const int i = so[t] + ex;
      if (i < so[t + 1]) {
        int n;
        if (same_rows(P.nch[i] * nx, n)) {
          rows = n;
          load_rows(m, P.AtR, (IX)P.fc[i] * (nx * nx) + ox, n, nx);
        }
      }
    };
    auto stage_b = [&](int t, S(&m)[kPre], int& rows) {
      if (t < 1) return;
      bool first = true;
      each_x(so[t], so[t + 1], [&](int i, int o, IX e) {
        const int fc = P.fc[i];
        const IX off = (IX)fc * (nx * nx) + o;
        const S* qc = qx + (size_t)fc * nx;
        const int n = __builtin_amdgcn_readfirstlane(rows);
        qx[e] += first && n > 0 ? dot_rows(m, P.AtR, off, n, nx, qc) : dot_n(P.AtR, off, P.nch[i] * nx, nx, qc);
        first = false;
      });
      fetch_b(t - 2, m, rows);
      stage_barrier();
    };
    fetch_b(N - 1, m0, r0);
    fetch_b(N - 2, m1, r1);
    __syncthreads();
    for (int t = N - 1; t >= 1; t -= 2) {
      stage_b(t, m0, r0);
      stage_b(t - 1, m1, r1);
    }
    // ---- mid: d, then what the children's states need of it
    each_u(0, P.nl, [&](int i, int o, IX e) {
      const int fc = P.fc[i];
      dd[e] = dot_u(P.Rinv, (IX)i * (nu * nu) + o, 0, nu, nu, uu + (size_t)i * nu) +
              dot_n(P.BtR, (IX)fc * (nx * nu) + o, P.nch[i] * nx, nu, qx + (size_t)fc * nx);
    });
    stage_barrier();
    each_x(1, P.nn, [&](int c, int o, IX e) {
      qx[e] = dot_u(P.BC, (IX)c * (nu * nx) + o, 0, nu, nx, dd + (size_t)P.anc[c] * nu);
    });
    if ((int)threadIdx.x < nx) qx[threadIdx.x] = (S)x0[threadIdx.x];
    // ---- forward chain
    auto fetch_f = [&](int t, S(&m)[kPre]) {
      if (t >= N) return;
      const int c = so[t + 1] + ex;
      if (c < so[t + 2]) load_rows(m, P.AbC, (IX)c * (nx * nx) + ox, nx, nx);
    };
    auto stage_f = [&](int t, S(&m)[kPre]) {
      if (t >= N) return;
      bool first = true;
      each_x(so[t + 1], so[t + 2], [&](int c, int o, IX e) {
        const IX off = (IX)c * (nx * nx) + o;
        const S* xi = qx + (size_t)P.anc[c] * nx;
        qx[e] += first ? dot_rows(m, P.AbC, off, nx, nx, xi) : dot_u(P.AbC, off, 0, nx, nx, xi);
        first = false;
      });
      fetch_f(t + 2, m);
      stage_barrier();
    };
    fetch_f(0, m0);
    fetch_f(1, m1);
    stage_barrier();
    for (int t = 0; t < N; t += 2) {
      stage_f(t, m0);
      stage_f(t + 1, m1);
    }
    // ---- post
    each_u(0, P.nl, [&](int i, int o, IX e) {
      const S up = dd[e] + dot_u(P.KC, (IX)i * (nx * nu) + o, 0, nx, nu, qx + (size_t)i * nx);
      dd[e] = up;
      at<S, IX>(zout, (IX)P.zU + e) = up;
    });
    for (IX e = threadIdx.x; e < (IX)P.nn * nx; e += kBT) at<S, IX>(zout, 1 + e) = qx[e];
    __syncthreads();
    StatAcc st;
    for (int i = team; i < P.nl; i += kTeams) {
      const S* xi = qx + (size_t)i * nx;
      const S* ui = dd + (size_t)i * nu - nx;
      flat_family<S, T, SL, IX>(P, O, O.s(i), z, eta, zout, eout, i, P.fc[i], P.nch[i], lane,
                                [&](int k) { return k < nx ? xi[k] : ui[k]; }, st);
    }
    for (int j = P.nl + team; j < P.nn; j += kTeams) {
      const S* xj = qx + (size_t)j * nx;
      flat_leaf<S, T, SL, IX>(P, O, O.s(j), z, eta, zout, eout, j, lane, [&](int k) { return xj[k]; }, st);
    }
    double o[5] = {st.rz2, st.re2, st.cross, st.xip, st.xid};
    blk_reduce<5, true>(o, red);  // its barriers also end the stores of T(v)
    BStats r;
    r.xip = o[3];
    r.xid = o[4];
    r.om2 = o[0] + o[1] - 2.0 * (double)P.alpha * o[2];
    return r;
  }

  // f(e, ...) over the vectors: out_k[e] = f(in_0[e], in_1[e], ...), 16 bytes
  // at a time, then the tail
  template <int NI, int NO, typename F>
  __device__ void map(const S* const (&in)[NI], S* const (&out)[NO], F&& f) const {
    const long long nw = nv / W;
    for (long long k = threadIdx.x; k < nw; k += kBT) {
      Vec16<S> x[NI], y[NO];
#pragma unroll
      for (int j = 0; j < NI; ++j) x[j] = reinterpret_cast<const Vec16<S>*>(in[j])[k];
#pragma unroll
      for (int q = 0; q < W; ++q) {
        S a[NI], b[NO];
#pragma unroll
        for (int j = 0; j < NI; ++j) a[j] = x[j].e[q];
        f(a, b);
#pragma unroll
        for (int j = 0; j < NO; ++j) y[j].e[q] = b[j];
      }
#pragma unroll
      for (int j = 0; j < NO; ++j) reinterpret_cast<Vec16<S>*>(out[j])[k] = y[j];
    }
    for (long long e = nw * W + threadIdx.x; e < nv; e += kBT) {
      S a[NI], b[NO];
#pragma unroll
      for (int j = 0; j < NI; ++j) a[j] = in[j][e];
      f(a, b);
#pragma unroll
      for (int j = 0; j < NO; ++j) out[j][e] = b[j];
    }
    __syncthreads();
  }

  // In FP32 the columns dV and dR stay apart and the direction subtracts them
  // in FP64: v and r change little from one iterate to the next, so both are
  // mostly exact, and so is dV - dR, which FP32 would round (1 to 2% of an
  // iteration). In FP64 the column E = dV - dR has the same bits either way.
  static constexpr bool kApart = sizeof(S) == 4;
  // Anderson push with MO older columns: r, dV (or E) and dR of the new column,
  // its Gram row and the right-hand side, then the solve
  template <int MO>
  __device__ void push(const S* v, const S* Tv, const S* vprev, const S* rprev, S* rcur, const AAPush& a, const AAPush* ap, double* G,
                       double* gamma, AARingDev* ring) const {
    const S* in[4 + MO];
    in[0] = v;
    in[1] = Tv;
    in[2] = vprev;
    in[3] = rprev;
#pragma unroll
    for (int j = 0; j < MO; ++j) in[4 + j] = pool(10 + kAAMax + a.order_old[j]);
    S* out[3] = {rcur, pool(10 + a.slot), pool(10 + kAAMax + a.slot)};
    double acc[2 * MO + 2];
#pragma unroll
    for (int j = 0; j < 2 * MO + 2; ++j) acc[j] = 0;
    map<4 + MO, 3>(in, out, [&](const S(&x)[4 + MO], S(&y)[3]) {
      const S r = x[0] - x[1], dr = r - x[3];
      y[0] = r;
      y[1] = kApart ? x[0] - x[2] : (x[0] - x[2]) - dr;
      y[2] = dr;
#pragma unroll
      for (int j = 0; j < MO; ++j) {
        acc[j] += (double)x[4 + j] * (double)dr;
        acc[MO + 1 + j] += (double)x[4 + j] * (double)r;
      }
      acc[MO] += (double)dr * (double)dr;
      acc[2 * MO + 1] += (double)dr * (double)r;
    });
    blk_reduce<2 * MO + 2, false>(acc, red);
    if (threadIdx.x == 0) {
#pragma unroll
      for (int j = 0; j < 2 * MO + 2; ++j) gamma[kAAMax + j] = acc[j];
      blk_gram_solve<MO>(G, gamma + kAAMax, ap, gamma, ring);
    }
    __syncthreads();
  }

  // Alg. 3 (or CP) as a state machine: one evaluation of T per trip
  __device__ void run(double* out) {
    enum { kInit, kCP, kK0, kLS, kK2, kKM };
    __shared__ double G[kAAMax * kAAMax], gamma[kAAMax + 8];  // gamma, then the push's dots
    __shared__ AARingDev ring;
    __shared__ AAPush next;
    S* v = pool(0);
    S* Tv = pool(1);
    S* vprev = pool(2);
    S* rprev = pool(3);
    S* rcur = pool(4);
    S* dir = pool(5);
    S* Md = pool(6);
    S* vt = pool(7);
    S* Tvt = pool(8);
    S* spare = pool(9);
    // Anderson columns of slot j: dV (or E) at pool(10 + j), dR at pool(10 + kAAMax + j)
    // x0 must lie in the root's state box
    bool box_ok = true;
    for (int o = 0; o < P.nx; ++o) box_ok = box_ok && x0[o] >= (double)P.xlo[o] && x0[o] <= (double)P.xhi[o];
    int status = box_ok ? -1 : 3, k = 0, n_k0 = 0, n_k1 = 0, n_k2 = 0, n_km = 0, n_bt = 0, t_evals = 0;
    double xi0 = 0, xi = 0, tol = 0, zeta = 0, omega_safe = 0, omega = 0, tau = 1.0;
    int ph = kInit, ls = 0;
    bool have_prev = false;
    BStats Sc;
    if (box_ok) {
      for (long long e = threadIdx.x; e < nv; e += kBT) v[e] = vio[e];
      if (threadIdx.x == 0) {
        ring = AARingDev{};
        ring.m = s.m;
      }
      __syncthreads();
    }
    auto rotate = [&](S*& point) {  // the accepted iterate and residual become the previous ones
      S* t1 = vprev;
      vprev = v;
      v = point;
      point = t1;
      S* t2 = rprev;
      rprev = rcur;
      rcur = t2;
      have_prev = true;
    };
    while (status < 0) {
      const bool line = ph == kLS;
      const BStats St = Teval(line ? vt : v, line ? Tvt : Tv);
      ++t_evals;
      if (line) {
        bool backtrack = !St.ok();
        if (!backtrack) {
          const double om_t = St.omega();
          if (om_t == 0.0 || (omega <= omega_safe && om_t <= s.c1 * omega)) {  // K1
            rotate(vt);
            S* t3 = Tv;
            Tv = Tvt;
            Tvt = t3;
            Sc = St;
            omega_safe = om_t + pow(s.c2, (double)k);
            ++n_k1;
          } else {
            double rd[1] = {0};
            for (long long e = threadIdx.x; e < nv; e += kBT)
              rd[0] += ((double)vt[e] - (double)Tvt[e]) * (double)Md[e];
            blk_reduce<1, false>(rd, red);
            const double rho = om_t * om_t - tau * rd[0];
            if (rho >= s.sigma * om_t * omega) {  // K2: v - c (vt - T vt)
              const double c = s.lambda * rho / (om_t * om_t);
              const S* in[3] = {v, vt, Tvt};
              S* o1[1] = {spare};
              map<3, 1>(in, o1, [&](const S(&x)[3], S(&y)[1]) {
                y[0] = (S)((double)x[0] + -c * (double)x[1] + c * (double)x[2]);
              });
              rotate(spare);
              ++n_k2;
              ph = kK2;
              continue;
            }
            backtrack = true;
          }
        }
        if (backtrack) {
          tau *= s.beta;
          ++n_bt;
          const bool again = ++ls < s.max_ls;
          // v + tau d, or the plain KM step v - lambda r
          const S* in[2] = {v, again ? dir : rcur};
          S* o1[1] = {again ? vt : spare};
          const double c = again ? tau : -s.lambda;
          map<2, 1>(in, o1, [&](const S(&x)[2], S(&y)[1]) { y[0] = (S)((double)x[0] + c * (double)x[1]); });
          if (!again) {
            rotate(spare);
            ++n_km;
            ph = kKM;
          }
          continue;
        }
        ++k;
      } else {
        Sc = St;
        if (ph == kInit) {
          xi0 = St.xi();
          tol = fmax(s.eps_abs, s.eps_rel * xi0);
          zeta = omega_safe = St.omega();
        } else {
          ++k;
        }
        if (!St.ok()) {
          status = 2;
          break;
        }
      }
      // ---- top of an iteration of Alg. 3
      if (Sc.xi() <= tol) {
        status = 0;
        break;
      }
      if (k >= s.max_iters) {
        status = 1;
        break;
      }
      if (s.method == SPOCK_METHOD_CP) {
        S* t1 = v;
        v = Tv;
        Tv = t1;
        ph = kCP;
        continue;
      }
      // residual r = v - T(v), the Anderson push and its Gram solve
      int dk = 0;
      double g[kAAMax] = {0, 0, 0, 0};
      const S *dV[kAAMax], *dR[kAAMax];
#pragma unroll
      for (int j = 0; j < kAAMax; ++j) dV[j] = dR[j] = rcur;
      if (have_prev) {
        if (threadIdx.x == 0) next = aa_next_push(&ring);
        __syncthreads();
        const AAPush& a = next;
        switch (a.mo) {
          case 0: push<0>(v, Tv, vprev, rprev, rcur, a, &next, G, gamma, &ring); break;
          case 1: push<1>(v, Tv, vprev, rprev, rcur, a, &next, G, gamma, &ring); break;
          case 2: push<2>(v, Tv, vprev, rprev, rcur, a, &next, G, gamma, &ring); break;
          default: push<3>(v, Tv, vprev, rprev, rcur, a, &next, G, gamma, &ring); break;
        }
        dk = ring.dk;
#pragma unroll
        for (int j = 0; j < kAAMax; ++j)
          if (j < dk) {
            g[j] = gamma[j];
            dV[j] = pool(10 + ring.dslot[j]);
            if (kApart) dR[j] = pool(10 + kAAMax + ring.dslot[j]);
          }
      } else {
        const S* in[2] = {v, Tv};
        S* o1[1] = {rcur};
        map<2, 1>(in, o1, [&](const S(&x)[2], S(&y)[1]) { y[0] = (S)((double)x[0] - (double)x[1]); });
      }
      omega = Sc.omega();
      const bool k0 = omega <= s.c0 * zeta;
      // d = -r - sum_j gamma_j (dV_j - dR_j) and the next point v + d (the K0 step, or
      // the first candidate of the line search, which keeps d as well)
      auto direction = [&](auto DK) {
        constexpr int D = decltype(DK)::value;
        constexpr int NI = 2 + (kApart ? 2 * D : D);
        const S* in[NI];
        in[0] = rcur;
        in[1] = v;
#pragma unroll
        for (int j = 0; j < D; ++j) {
          in[2 + j] = dV[j];
          if (kApart) in[NI - D + j] = dR[j];
        }
        auto one = [&](const S(&x)[NI]) {
          double acc = -(double)x[0];
#pragma unroll
          for (int j = 0; j < D; ++j) acc -= g[j] * ((double)x[2 + j] - (kApart ? (double)x[NI - D + j] : 0.0));
          return (S)acc;
        };
        if (k0) {
          S* o1[1] = {spare};
          map<NI, 1>(in, o1, [&](const S(&x)[NI], S(&y)[1]) { y[0] = (S)((double)x[1] + (double)one(x)); });
        } else {
          S* o2[2] = {vt, dir};
          map<NI, 2>(in, o2, [&](const S(&x)[NI], S(&y)[2]) {
            y[1] = one(x);
            y[0] = (S)((double)x[1] + (double)y[1]);
          });
        }
      };
      switch (dk) {
        case 0: direction(std::integral_constant<int, 0>{}); break;
        case 1: direction(std::integral_constant<int, 1>{}); break;
        case 2: direction(std::integral_constant<int, 2>{}); break;
        case 3: direction(std::integral_constant<int, 3>{}); break;
        default: direction(std::integral_constant<int, 4>{}); break;
      }
      if (k0) {
        rotate(spare);
        zeta = omega;
        ++n_k0;
        ph = kK0;
        continue;
      }
      for (int i = team; i < P.nl; i += kTeams) fam_apply_M<S, T>(P, dir, Md, i, lane);
      __syncthreads();
      tau = 1.0;
      ls = 0;
      ph = kLS;
    }
    if (box_ok) {
      xi = Sc.xi();
      for (long long e = threadIdx.x; e < nv; e += kBT) vio[e] = Tv[e];
      if (threadIdx.x == 0) out[8] = (double)Tv[0];
    }
    if (threadIdx.x == 0) {
      out[0] = status;
      out[1] = k;
      out[2] = t_evals;
      out[3] = n_k0;
      out[4] = n_k1;
      out[5] = n_k2;
      out[6] = n_km;
      out[7] = n_bt;
      out[9] = xi0;
      out[10] = xi;
    }
  }
};

template <typename S, int T, int SL, bool LQ>
__global__ void __launch_bounds__(kBT) k_solve_batched(const BatchInst<S>* __restrict__ insts, BatchSettings s, BLds L,
                                                       double* __restrict__ infos) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[8 * kBW];
  BlockSolver<S, T, SL, LQ> solver(insts[blockIdx.x], s, smem_raw, L, red);
  solver.run(infos + (size_t)insts[blockIdx.x].id * 16);
}

template <typename S, int T, int SL, bool LQ>
hipError_t launch_form(const BatchInst<S>* insts, int B, const BatchSettings& s, const BLds& L, double* infos,
                       hipStream_t st) {
  const int lds = LQ ? (int)L.total : 0;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_solve_batched<S, T, SL, LQ>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((k_solve_batched<S, T, SL, LQ>), dim3(B), dim3(kBT), lds, st, insts, s, L, infos);
  return hipGetLastError();
}
template <typename S, int T, int SL>
hipError_t launch_team(const BatchInst<S>* insts, int B, const BatchSettings& s, const BLds& L, double* infos,
                       hipStream_t st) {
  // the exchange buffers in LDS when the largest tree fits
  return L.total <= kBLds ? launch_form<S, T, SL, true>(insts, B, s, L, infos, st)
                          : launch_form<S, T, SL, false>(insts, B, s, L, infos, st);
}

}  // namespace

template <typename S>
hipError_t launch_solve_batched(const BatchInst<S>* insts_dev, int B, const BatchSettings& s, int team,
                                const BatchShape& sh, double* infos_dev, hipStream_t st) {
  const BLds L = blk_lds(sizeof(S), sh);
  switch (team) {
    case 8: return launch_team<S, 8, 1>(insts_dev, B, s, L, infos_dev, st);
    case 16: return launch_team<S, 16, 1>(insts_dev, B, s, L, infos_dev, st);
    case 32: return launch_team<S, 32, 1>(insts_dev, B, s, L, infos_dev, st);
    default: return sh.nx + sh.nu <= 64 ? launch_team<S, 64, 1>(insts_dev, B, s, L, infos_dev, st)
                                        : launch_team<S, 64, 2>(insts_dev, B, s, L, infos_dev, st);
  }
}
template hipError_t launch_solve_batched<double>(const BatchInst<double>*, int, const BatchSettings&, int,
                                                 const BatchShape&, double*, hipStream_t);
template hipError_t launch_solve_batched<float>(const BatchInst<float>*, int, const BatchSettings&, int,
                                                const BatchShape&, double*, hipStream_t);

size_t batched_work_elems(int nn, int nl, int nx, int nu, long long nv) {
  return (size_t)kBPool * (size_t)((nv + 63) & ~63LL) + (size_t)nn * nx + 2 * (size_t)nl * nu;
}

}  // namespace spk
