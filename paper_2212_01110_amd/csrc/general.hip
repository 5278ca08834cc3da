// Kernels of general problems: a conic risk measure (E, F, b, K) at every
// nonleaf node (section 4.3) and polyhedral constraints Gamma_x x + Gamma_u u
// in C (section 4.1, eq. constraints) in place of AV@R and the boxes. Only
// the parts of T that touch y, the constraint rows and the leaves' rows
// change; the Alg. 2 sweeps are shared with every other problem.
//
// One wavefront per unit. The units are the families (nonleaf node i: group 1
// of i, group 2 of each child; columns y^i, s^i, x^i, u^i, tau of each child)
// and the leaves (group 3; columns x^j, s^j): every row of L and every column
// of L* belongs to exactly one unit, so no unit waits on another. Lane o owns
// component o of every state and input (n_x, n_u <= 64); constraint rows go 64
// at a time, one lane a row, with the row values left in LDS for the columns.
// The kernels are bound by the latency of a unit's load chains (a unit's data
// is a few KiB): one thread per family walked every row and column alone, 372
// and 115 us for the post- and pre-pass of a 364-node tree (n_x 13, n_u 6, 9
// and 7 rows, FP64) that move 0.5 MB.
#include "device_common.h"

#include <math.h>
#include <algorithm>

namespace spk {

namespace {

constexpr int kGenThreads = 256;
constexpr int kGenWaves = kGenThreads / 64;

// Offsets in the general layout.
template <typename S>
struct GOff {
  const DevProb<S>& P;
  const GenDev<S>& G;
  __device__ GOff(const DevProb<S>& p, const GenDev<S>& g) : P(p), G(g) {}
  __device__ long long x(int i) const { return 1 + (long long)i * P.nx; }
  __device__ long long u(int i) const { return P.zU + (long long)i * P.nu; }
  __device__ long long y(int i) const { return G.z2off[i]; }
  __device__ long long tau(int c) const {
    const int a = P.anc[c];
    return G.z2off[a] + G.ny[a] + (c - P.fc[a]);
  }
  __device__ long long s(int c) const {
    if (c == 0) return 0;
    const int a = P.anc[c];
    return G.z2off[a] + G.ny[a] + P.nch[a] + (c - P.fc[a]);
  }
  __device__ long long e1(int i) const { return G.e1off[i]; }
  __device__ long long e1s(int i) const { return G.e1off[i] + G.ny[i]; }
  __device__ long long e1c(int i) const { return e1s(i) + 1; }
  __device__ long long e2(int c) const { return G.eE2 + (long long)(c - 1) * (P.nx + P.nu + 2); }
  __device__ long long e3(int j) const { return G.eE3 + (long long)(j - P.nl) * (G.ncN + P.nx + 2); }
  __device__ long long e3q(int j) const { return e3(j) + G.ncN; }
  __device__ const S* Gx(int i) const { return G.Gx + (size_t)i * G.nc * P.nx; }
  __device__ const S* Gu(int i) const { return G.Gu + (size_t)i * G.nc * P.nu; }
  __device__ const S* GN(int j) const { return G.GN + (size_t)(j - P.nl) * G.ncN * P.nx; }
  __device__ const S* root(int kind) const { return kind == 0 ? G.Qh : (kind == 1 ? G.Rh : G.QNh); }
  // Component o of a cost root of node c applied to a vector: kind 0 Q^c (on
  // x), 1 R^c (on u), 2 Q_N^c (on x). Diagonal roots scale the lane's own
  // component; dense ones (symmetric, so the columns are read: lane o at
  // k n + o, coalesced) need the whole vector at vec (LDS or global). The
  // same columns give the L* columns.
  __device__ S croot(int kind, int c, int o, S own, const S* vec) const {
    const int n = kind == 1 ? P.nu : P.nx;
    const S* M = root(kind);
    if (M) {
      const S* col = M + (size_t)c * n * n + o;
      S acc = 0;
#pragma unroll 4
      for (int k = 0; k < n; ++k) acc += col[(size_t)k * n] * vec[k];
      return acc;
    }
    const S* dg = kind == 0 ? P.sq : (kind == 1 ? P.sr : P.sqN);
    return dg[(size_t)c * n + o] * own;
  }
};

// sum_r M[r][o] v[r], r < rows (M row-major with ld columns): lane o's column
template <typename S>
__device__ __forceinline__ S col_dot(const S* __restrict__ M, int rows, int ld, int o, const S* v, S acc) {
#pragma unroll 8
  for (int r = 0; r < rows; ++r) acc += M[(size_t)r * ld + o] * v[r];
  return acc;
}
// sum_o row[o] v[o], o < n: one lane per row
template <typename S>
__device__ __forceinline__ S row_dot(const S* __restrict__ row, int n, const S* v, S acc) {
#pragma unroll 8
  for (int o = 0; o < n; ++o) acc += row[o] * v[o];
  return acc;
}

// (L* eta) on columns x^i (or u^i) of nonleaf i, component o: Gamma' eta_c
// plus the children's cost-root rows.
template <typename S>
__device__ __forceinline__ S lt_x(const GOff<S>& O, const S* eta, int i, int o) {
  const DevProb<S>& P = O.P;
  S acc = col_dot(O.Gx(i), O.G.nc, P.nx, o, eta + O.e1c(i), S(0));
  for (int c = P.fc[i]; c < P.fc[i] + P.nch[i]; ++c) acc += O.croot(0, c, o, eta[O.e2(c) + o], eta + O.e2(c));
  return acc;
}
template <typename S>
__device__ __forceinline__ S lt_u(const GOff<S>& O, const S* eta, int i, int o) {
  const DevProb<S>& P = O.P;
  S acc = col_dot(O.Gu(i), O.G.nc, P.nu, o, eta + O.e1c(i), S(0));
  for (int c = P.fc[i]; c < P.fc[i] + P.nch[i]; ++c) {
    const long long e = O.e2(c) + P.nx;
    acc += O.croot(1, c, o, eta[e + o], eta + e);
  }
  return acc;
}
// column x^j of leaf j: Gamma_N' eta_cN + Q_N^{1/2} eta_q
template <typename S>
__device__ __forceinline__ S lt_xleaf(const GOff<S>& O, const S* eta, int j, int o) {
  const long long e3q = O.e3q(j);
  return col_dot(O.GN(j), O.G.ncN, O.P.nx, o, eta + O.e3(j), O.croot(2, j, o, eta[e3q + o], eta + e3q));
}
// column s^c: the s-row of c when c is nonleaf, else half the sum of its
// group-3 pair
template <typename S>
__device__ __forceinline__ S lt_s(const GOff<S>& O, const S* eta, int c) {
  if (c < O.P.nl) return eta[O.e1s(c)];
  const long long e = O.e3q(c) + O.P.nx;
  return S(0.5) * (eta[e] + eta[e + 1]);
}

// prox of g* of one unit for the dual argument at w (rows as in eta), written
// to out (which may be w): group 1 (K* on y, R_+ on the s-row, C^i on the
// constraint rows) and group 2 of every child of a family, or group 3 of a
// leaf.
template <typename S>
__device__ void unit_gen_prox(const GOff<S>& O, const S* w, S* out, int i, int lane) {
  const DevProb<S>& P = O.P;
  const GenDev<S>& G = O.G;
  const int nx = P.nx, nu = P.nu;
  const S al = P.alpha, ia = S(1) / al;
  const bool onx = lane < nx, onu = lane < nu;
  if (i < P.nl) {
    const long long e1 = O.e1(i), ec = O.e1c(i);
    const int ny = G.ny[i], kp = G.kpos[i];
    for (int k = lane; k <= ny; k += 64) {  // y, then the s-row
      const S v = w[e1 + k];
      out[e1 + k] = (k < kp || k == ny) ? (v < S(0) ? v : S(0)) : S(0);
    }
    for (int r = lane; r < G.nc; r += 64) {
      const S v = w[ec + r];
      out[ec + r] = v - al * clampv(v * ia, G.cmin[(size_t)i * G.nc + r], G.cmax[(size_t)i * G.nc + r]);
    }
    for (int c = P.fc[i]; c < P.fc[i] + P.nch[i]; ++c) {
      const long long e2 = O.e2(c);
      S wx = onx ? w[e2 + lane] : S(0), wu = onu ? w[e2 + nx + lane] : S(0);
      S wa = w[e2 + nx + nu], wb = w[e2 + nx + nu + 1];
      soc_prox_wave(wx, onx, wu, onu, wa, wb, al);
      if (onx) out[e2 + lane] = wx;
      if (onu) out[e2 + nx + lane] = wu;
      if (lane == 0) {
        out[e2 + nx + nu] = wa;
        out[e2 + nx + nu + 1] = wb;
      }
    }
    return;
  }
  const long long e3 = O.e3(i), e3q = O.e3q(i);
  const size_t lj = (size_t)(i - P.nl) * G.ncN;
  for (int r = lane; r < G.ncN; r += 64) {
    const S v = w[e3 + r];
    out[e3 + r] = v - al * clampv(v * ia, G.cNmin[lj + r], G.cNmax[lj + r]);
  }
  S wx = onx ? w[e3q + lane] : S(0), none = S(0);
  S wa = w[e3q + nx], wb = w[e3q + nx + 1];
  soc_prox_wave(wx, onx, none, false, wa, wb, al);
  if (onx) out[e3q + lane] = wx;
  if (lane == 0) {
    out[e3q + nx] = wa;
    out[e3q + nx + 1] = wb;
  }
}

// rows of L z of one unit, written into eta (or, with base, eta = base + scale L z)
template <typename S>
__device__ void unit_gen_L(const GOff<S>& O, const S* z, S* eta, int i, const S* base, S scale, int lane) {
  const DevProb<S>& P = O.P;
  const GenDev<S>& G = O.G;
  const int nx = P.nx, nu = P.nu;
  const bool onx = lane < nx, onu = lane < nu;
  auto put = [&](long long e, S v) { eta[e] = base ? base[e] + scale * v : v; };
  const S* xi = z + O.x(i);
  if (i < P.nl) {
    const long long e1 = O.e1(i), zy = O.y(i);
    const int ny = G.ny[i];
    const S* b = G.b + G.yoff[i];
    double by = 0;
    for (int k = lane; k < ny; k += 64) {
      const S y = z[zy + k];
      put(e1 + k, y);
      by += (double)(b[k] * y);
    }
    by = team_sum<64>(by);
    if (lane == 0) put(O.e1s(i), (S)((double)z[O.s(i)] - by));
    const S* ui = z + O.u(i);
    for (int r = lane; r < G.nc; r += 64)
      put(O.e1c(i) + r,
          row_dot(O.Gu(i) + (size_t)r * nu, nu, ui, row_dot(O.Gx(i) + (size_t)r * nx, nx, xi, S(0))));
    for (int c = P.fc[i]; c < P.fc[i] + P.nch[i]; ++c) {
      const long long e2 = O.e2(c);
      if (onx) put(e2 + lane, O.croot(0, c, lane, xi[lane], xi));
      if (onu) put(e2 + nx + lane, O.croot(1, c, lane, ui[lane], ui));
      if (lane < 2) put(e2 + nx + nu + lane, S(0.5) * z[O.tau(c)]);
    }
    return;
  }
  const long long e3 = O.e3(i), e3q = O.e3q(i);
  for (int r = lane; r < G.ncN; r += 64) put(e3 + r, row_dot(O.GN(i) + (size_t)r * nx, nx, xi, S(0)));
  if (onx) put(e3q + lane, O.croot(2, i, lane, xi[lane], xi));
  if (lane < 2) put(e3q + nx + lane, S(0.5) * z[O.s(i)]);
}

// columns of L* eta of one unit, written into z (or, with base, z = base + scale L* eta)
template <typename S>
__device__ void unit_gen_Lt(const GOff<S>& O, const S* eta, S* z, int i, const S* base, S scale, int lane) {
  const DevProb<S>& P = O.P;
  const GenDev<S>& G = O.G;
  const int nx = P.nx, nu = P.nu;
  const bool onx = lane < nx, onu = lane < nu;
  auto put = [&](long long e, S v) { z[e] = base ? base[e] + scale * v : v; };
  if (i < P.nl) {
    const S es = eta[O.e1s(i)];
    const S* b = G.b + G.yoff[i];
    for (int k = lane; k < G.ny[i]; k += 64) put(O.y(i) + k, eta[O.e1(i) + k] - b[k] * es);
    if (lane == 0) put(O.s(i), es);
    if (onx) put(O.x(i) + lane, lt_x<S>(O, eta, i, lane));
    if (onu) put(O.u(i) + lane, lt_u<S>(O, eta, i, lane));
    for (int k = lane; k < P.nch[i]; k += 64) {
      const int c = P.fc[i] + k;
      const long long e2 = O.e2(c) + nx + nu;
      put(O.tau(c), S(0.5) * (eta[e2] + eta[e2 + 1]));
    }
    return;
  }
  if (onx) put(O.x(i) + lane, lt_xleaf<S>(O, eta, i, lane));
  if (lane == 0) put(O.s(i), lt_s<S>(O, eta, i));
}

// ---------------------------------------------------------------- kernels
// pre-pass of T: xbar, ubar = (x, u) - alpha L* eta; leaves seed the backward
// sweep with q = -xbar; the (y, tau, s) block of the step z - alpha L* eta is
// projected on S2 (kernel of [E' -I -I; F' 0 0], the projector formed
// offline; symmetric, so lane r reads column r); s^0 - alpha at the root.
template <typename S>
__global__ void __launch_bounds__(kGenThreads) k_gen_pre(DevProb<S> P, GenDev<S> G, const S* __restrict__ z,
                                                       const S* __restrict__ eta, S* __restrict__ zout,
                                                       S* __restrict__ xbar, S* __restrict__ ubar,
                                                       S* __restrict__ qbuf) {
  __shared__ S wsh[kGenWaves][kGenMaxBlock];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = blockIdx.x * kGenWaves + wave;
  if (i >= P.nn) return;  // whole wavefronts only; no block barrier below
  const GOff<S> O(P, G);
  const int nx = P.nx, nu = P.nu;
  const S al = P.alpha;
  if (i >= P.nl) {
    if (lane < nx) qbuf[(size_t)i * nx + lane] = -(z[O.x(i) + lane] - al * lt_xleaf<S>(O, eta, i, lane));
    return;
  }
  const int fc = P.fc[i], n = P.nch[i], ny = G.ny[i];
  // the (y, tau, s) block after the step
  S* w = wsh[wave];
  const S es = eta[O.e1s(i)];
  const S* b = G.b + G.yoff[i];
  const long long zb = O.y(i);
  for (int k = lane; k < ny; k += 64) w[k] = z[zb + k] - al * (eta[O.e1(i) + k] - b[k] * es);
  for (int k = lane; k < n; k += 64) {
    const int c = fc + k;
    const long long e2 = O.e2(c) + nx + nu;
    w[ny + k] = z[zb + ny + k] - al * S(0.5) * (eta[e2] + eta[e2 + 1]);
    w[ny + n + k] = z[zb + ny + n + k] - al * lt_s<S>(O, eta, c);
  }
  if (lane < nx) xbar[(size_t)i * nx + lane] = z[O.x(i) + lane] - al * lt_x<S>(O, eta, i, lane);
  if (lane < nu) ubar[(size_t)i * nu + lane] = z[O.u(i) + lane] - al * lt_u<S>(O, eta, i, lane);
  if (i == 0 && lane == 0) zout[0] = z[0] - al * es - al;
  wave_lds_sync();
  const int m = ny + 2 * n;
  const S* Pm = G.PS2 + G.Poff[i];
  for (int r = lane; r < m; r += 64) zout[zb + r] = col_dot(Pm, m, m, r, w, S(0));
}

// post-pass of T: eta+ = prox_{alpha g*}(eta + alpha L (2 z+ - z)) on the
// unit's rows, and the residual statistics of r = v - T(v) on its rows
// (||r_eta||^2, <r_eta, L r_z>, |r_eta / alpha - L r_z|) and columns
// (||r_z||^2, |r_z / alpha - L* r_eta|). Grid-stride over units, one record
// per block. LDS per wavefront: 2 z+ - z and r_z of (x, u), and the r_eta of
// 64 constraint rows or of a cone block (dense roots read it whole).
template <typename S>
__global__ void __launch_bounds__(kGenThreads) k_gen_post(DevProb<S> P, GenDev<S> G, const S* __restrict__ z,
                                                        const S* __restrict__ eta, const S* __restrict__ zout,
                                                        S* __restrict__ eout, double* __restrict__ partials) {
  __shared__ S lds[kGenWaves][6][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  S* X2 = lds[wave][0];
  S* U2 = lds[wave][1];
  S* RX = lds[wave][2];
  S* RU = lds[wave][3];
  S* E0 = lds[wave][4];
  S* E1 = lds[wave][5];
  const GOff<S> O(P, G);
  const int nx = P.nx, nu = P.nu;
  const bool onx = lane < nx, onu = lane < nu;
  const int ox = onx ? lane : 0, ou = onu ? lane : 0;
  const S al = P.alpha, sia = S(1) / al;
  const double ia = 1.0 / (double)al;
  StatAcc st;
  // one row: the argument's prox ep given, its r_eta against (L r_z)
  auto row = [&](long long e, S old, S ep, S Lrz) {
    eout[e] = ep;
    const S re = old - ep;
    st.row((double)re, (double)Lrz, ia);
    return re;
  };
  // rows of a constraint block (Gamma z in [lo, hi]), 64 at a time; their
  // part of the columns added to cx, cu (lane o: component o)
  auto cons = [&](int rows, long long ec, const S* gx, const S* gu, const S* lo, const S* hi, S& cx, S& cu) {
    for (int r0 = 0; r0 < rows; r0 += 64) {
      const int r = r0 + lane;
      wave_lds_sync();
      if (r < rows) {
        const S* rx = gx + (size_t)r * nx;
        S a2 = 0, ar = 0;
#pragma unroll 8
        for (int o = 0; o < nx; ++o) {
          a2 += rx[o] * X2[o];
          ar += rx[o] * RX[o];
        }
        if (gu) {
          const S* ru = gu + (size_t)r * nu;
#pragma unroll 8
          for (int o = 0; o < nu; ++o) {
            a2 += ru[o] * U2[o];
            ar += ru[o] * RU[o];
          }
        }
        const S old = eta[ec + r];
        const S w = old + al * a2;
        E0[lane] = row(ec + r, old, w - al * clampv(w * sia, lo[r], hi[r]), ar);
      }
      wave_lds_sync();
      const int m = rows - r0 < 64 ? rows - r0 : 64;
      if (onx) cx = col_dot(gx + (size_t)r0 * nx, m, nx, lane, E0, cx);
      if (gu && onu) cu = col_dot(gu + (size_t)r0 * nu, m, nu, lane, E0, cu);
    }
    wave_lds_sync();
  };
  for (int i = blockIdx.x * kGenWaves + wave; i < P.nn; i += gridDim.x * kGenWaves) {
    const long long xi = O.x(i);
    const S zx = z[xi + ox], zxp = zout[xi + ox];
    const S x2 = S(2) * zxp - zx, rx = zx - zxp;
    wave_lds_sync();  // the previous unit's readers are done
    if (onx) {
      X2[lane] = x2;
      RX[lane] = rx;
    }
    S cx = 0, cu = 0;  // (L* r_eta) on columns x^i, u^i
    if (i >= P.nl) {   // ---- a leaf: group 3, columns x^i, s^i
      wave_lds_sync();
      const long long e3 = O.e3(i), e3q = O.e3q(i), sp = O.s(i);
      const S s2 = S(2) * zout[sp] - z[sp], rs = z[sp] - zout[sp];
      const S oq = eta[e3q + ox], oa = eta[e3q + nx], ob = eta[e3q + nx + 1];
      S w = oq + al * O.croot(2, i, ox, x2, X2), none = S(0);
      const S lr = O.croot(2, i, ox, rx, RX);
      S wa = oa + al * S(0.5) * s2, wb = ob + al * S(0.5) * s2;
      soc_prox_wave(w, onx, none, false, wa, wb, al);
      S req = 0;
      if (onx) req = row(e3q + lane, oq, w, lr);
      if (lane == 0) {
        const S ra = row(e3q + nx, oa, wa, S(0.5) * rs), rb = row(e3q + nx + 1, ob, wb, S(0.5) * rs);
        st.col((double)rs, (double)(S(0.5) * (ra + rb)), ia);
      }
      if (onx) E1[lane] = req;
      wave_lds_sync();
      if (onx) cx = O.croot(2, i, lane, req, E1);
      const size_t lj = (size_t)(i - P.nl) * G.ncN;
      cons(G.ncN, e3, O.GN(i), nullptr, G.cNmin + lj, G.cNmax + lj, cx, cu);
      if (onx) st.col((double)rx, (double)cx, ia);
      continue;
    }
    const long long ui = O.u(i);
    const S zu = z[ui + ou], zup = zout[ui + ou];
    const S u2 = S(2) * zup - zu, ru = zu - zup;
    if (onu) {
      U2[lane] = u2;
      RU[lane] = ru;
    }
    wave_lds_sync();
    const int fc = P.fc[i], n = P.nch[i], ny = G.ny[i], kp = G.kpos[i];
    // ---- group 1: y in K*, s - b'y in R_+, the constraint rows; columns y^i, s^i
    const long long e1 = O.e1(i), zy = O.y(i), sp = O.s(i);
    const S* b = G.b + G.yoff[i];
    double by2 = 0, byr = 0;
    for (int k = lane; k < ny; k += 64) {
      const S y = z[zy + k], yp = zout[zy + k];
      by2 += (double)(b[k] * (S(2) * yp - y));
      byr += (double)(b[k] * (y - yp));
    }
    by2 = team_sum<64>(by2);
    byr = team_sum<64>(byr);
    const S s0 = z[sp], sp0 = zout[sp], es = eta[e1 + ny];
    const S ws = es + al * (S)((double)(S(2) * sp0 - s0) - by2);
    const S esn = ws < S(0) ? ws : S(0);
    const S res = es - esn;
    for (int k = lane; k < ny; k += 64) {
      const S y = z[zy + k], yp = zout[zy + k], old = eta[e1 + k];
      const S w = old + al * (S(2) * yp - y);
      const S re = row(e1 + k, old, k < kp ? (w < S(0) ? w : S(0)) : S(0), y - yp);
      st.col((double)(y - yp), (double)(re - b[k] * res), ia);
    }
    if (lane == 0) {
      row(e1 + ny, es, esn, (S)((double)(s0 - sp0) - byr));
      st.col((double)(s0 - sp0), (double)res, ia);
    }
    cons(G.nc, O.e1c(i), O.Gx(i), O.Gu(i), G.cmin + (size_t)i * G.nc, G.cmax + (size_t)i * G.nc, cx, cu);
    // ---- group 2 of every child: (Q^{1/2} x^i, R^{1/2} u^i, tau/2, tau/2); column tau
    for (int c = fc; c < fc + n; ++c) {
      const long long e2 = O.e2(c), tp = zy + ny + (c - fc);
      const S t2 = S(2) * zout[tp] - z[tp], rt = z[tp] - zout[tp];
      const S ex = eta[e2 + ox], eu = eta[e2 + nx + ou], ea = eta[e2 + nx + nu], eb = eta[e2 + nx + nu + 1];
      S wx = ex + al * O.croot(0, c, ox, x2, X2), wu = eu + al * O.croot(1, c, ou, u2, U2);
      const S lx = O.croot(0, c, ox, rx, RX), lu = O.croot(1, c, ou, ru, RU);
      S wa = ea + al * S(0.5) * t2, wb = eb + al * S(0.5) * t2;
      soc_prox_wave(wx, onx, wu, onu, wa, wb, al);
      S rex = 0, reu = 0;
      if (onx) rex = row(e2 + lane, ex, wx, lx);
      if (onu) reu = row(e2 + nx + lane, eu, wu, lu);
      if (lane == 0) {
        const S ra = row(e2 + nx + nu, ea, wa, S(0.5) * rt), rb = row(e2 + nx + nu + 1, eb, wb, S(0.5) * rt);
        st.col((double)rt, (double)(S(0.5) * (ra + rb)), ia);
      }
      if (onx) E0[lane] = rex;
      if (onu) E1[lane] = reu;
      wave_lds_sync();
      if (onx) cx += O.croot(0, c, lane, rex, E0);
      if (onu) cu += O.croot(1, c, lane, reu, E1);
      wave_lds_sync();
    }
    if (onx) st.col((double)rx, (double)cx, ia);
    if (onu) st.col((double)ru, (double)cu, ia);
  }
  // wavefront, then the block's wavefronts in order
  const double v[kStats] = {team_sum<64>(st.rz2), team_sum<64>(st.re2), team_sum<64>(st.cross), wave_max(st.xip),
                            wave_max(st.xid)};
  __shared__ double red[kGenWaves][kStats];
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < kStats; ++k) red[wave][k] = v[k];
  }
  __syncthreads();
  if (threadIdx.x < kStats) {
    const int k = threadIdx.x;
    double a = red[0][k];
    for (int w = 1; w < kGenWaves; ++w) a = (k < 3) ? a + red[w][k] : fmax(a, red[w][k]);
    partials[(size_t)blockIdx.x * kStats + k] = a;
  }
}

template <typename S>
__global__ void __launch_bounds__(kGenThreads) k_gen_L(DevProb<S> P, GenDev<S> G, const S* __restrict__ z,
                                                     S* __restrict__ eta) {
  const int i = blockIdx.x * kGenWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (i < P.nn) unit_gen_L<S>(GOff<S>(P, G), z, eta, i, nullptr, S(1), threadIdx.x & 63);
}
template <typename S>
__global__ void __launch_bounds__(kGenThreads) k_gen_Lt(DevProb<S> P, GenDev<S> G, const S* __restrict__ eta,
                                                      S* __restrict__ z) {
  const int i = blockIdx.x * kGenWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (i < P.nn) unit_gen_Lt<S>(GOff<S>(P, G), eta, z, i, nullptr, S(1), threadIdx.x & 63);
}
template <typename S>
__global__ void __launch_bounds__(kGenThreads) k_gen_prox_gstar(DevProb<S> P, GenDev<S> G, const S* w, S* out) {
  const int i = blockIdx.x * kGenWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (i < P.nn) unit_gen_prox<S>(GOff<S>(P, G), w, out, i, threadIdx.x & 63);
}
// M d = (d_z - alpha L* d_eta, d_eta - alpha L d_z)
template <typename S>
__global__ void __launch_bounds__(kGenThreads) k_gen_M(DevProb<S> P, GenDev<S> G, const S* __restrict__ d,
                                                     S* __restrict__ Md) {
  const int i = blockIdx.x * kGenWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (i >= P.nn) return;
  const GOff<S> O(P, G);
  unit_gen_Lt<S>(O, d + P.nz, Md, i, d, -P.alpha, threadIdx.x & 63);
  unit_gen_L<S>(O, d, Md + P.nz, i, d + P.nz, -P.alpha, threadIdx.x & 63);
}

template <typename S>
const GenDev<S>& gen_of(const Problem& P);
template <>
const GenDev<double>& gen_of<double>(const Problem& P) { return P.gd64; }
template <>
const GenDev<float>& gen_of<float>(const Problem& P) { return P.gd32; }
template <typename S>
const DevProb<S>& dev_of_g(const Problem& P);
template <>
const DevProb<double>& dev_of_g<double>(const Problem& P) { return P.dp64; }
template <>
const DevProb<float>& dev_of_g<float>(const Problem& P) { return P.dp32; }

int gen_blocks(const Problem& P) { return (P.tree->nn + kGenWaves - 1) / kGenWaves; }

}  // namespace

// one statistics record per block; the partials hold one per nonleaf node
// plus one, so wide families make the wavefronts loop
int gen_post_blocks(const Problem& P) { return std::max(1, std::min(gen_blocks(P), P.tree->nl + 1)); }

template <typename S>
hipError_t launch_gen_pre(const Problem& P, const S* z, const S* eta, S* zout, S* xbar, S* ubar, S* qbuf,
                          hipStream_t st) {
  hipLaunchKernelGGL(k_gen_pre<S>, dim3(gen_blocks(P)), dim3(kGenThreads), 0, st, dev_of_g<S>(P), gen_of<S>(P), z,
                     eta, zout, xbar, ubar, qbuf);
  return hipGetLastError();
}
template <typename S>
hipError_t launch_gen_post(const Problem& P, const S* z, const S* eta, const S* zout, S* eout, double* partials,
                           hipStream_t st) {
  hipLaunchKernelGGL(k_gen_post<S>, dim3(gen_post_blocks(P)), dim3(kGenThreads), 0, st, dev_of_g<S>(P), gen_of<S>(P),
                     z, eta, zout, eout, partials);
  return hipGetLastError();
}
template <typename S>
hipError_t launch_gen_L(const Problem& P, const S* z, S* eta, hipStream_t st) {
  hipLaunchKernelGGL(k_gen_L<S>, dim3(gen_blocks(P)), dim3(kGenThreads), 0, st, dev_of_g<S>(P), gen_of<S>(P), z,
                     eta);
  return hipGetLastError();
}
template <typename S>
hipError_t launch_gen_Lt(const Problem& P, const S* eta, S* z, hipStream_t st) {
  hipLaunchKernelGGL(k_gen_Lt<S>, dim3(gen_blocks(P)), dim3(kGenThreads), 0, st, dev_of_g<S>(P), gen_of<S>(P), eta,
                     z);
  return hipGetLastError();
}
template <typename S>
hipError_t launch_gen_prox_gstar(const Problem& P, const S* w, S* out, hipStream_t st) {
  hipLaunchKernelGGL(k_gen_prox_gstar<S>, dim3(gen_blocks(P)), dim3(kGenThreads), 0, st, dev_of_g<S>(P),
                     gen_of<S>(P), w, out);
  return hipGetLastError();
}
template <typename S>
hipError_t launch_gen_M(const Problem& P, const S* d, S* Md, hipStream_t st) {
  hipLaunchKernelGGL(k_gen_M<S>, dim3(gen_blocks(P)), dim3(kGenThreads), 0, st, dev_of_g<S>(P), gen_of<S>(P), d,
                     Md);
  return hipGetLastError();
}

#define SPK_GEN_INST(S)                                                                                    \
  template hipError_t launch_gen_pre<S>(const Problem&, const S*, const S*, S*, S*, S*, S*, hipStream_t);     \
  template hipError_t launch_gen_post<S>(const Problem&, const S*, const S*, const S*, S*, double*,          \
                                         hipStream_t);                                                     \
  template hipError_t launch_gen_L<S>(const Problem&, const S*, S*, hipStream_t);                           \
  template hipError_t launch_gen_Lt<S>(const Problem&, const S*, S*, hipStream_t);                          \
  template hipError_t launch_gen_prox_gstar<S>(const Problem&, const S*, S*, hipStream_t);                  \
  template hipError_t launch_gen_M<S>(const Problem&, const S*, S*, hipStream_t);
SPK_GEN_INST(double)
SPK_GEN_INST(float)

}  // namespace spk
