// Kernels of the implicit differentiation at the fixed point v* = T(v*):
// the Jacobian of prox_{alpha g*} at the pre-prox point b* (section 5.4:
// G(b) = b - alpha proj_S3(b / alpha), so J_G = I - J_proj(b* / alpha)),
// the transpose of the root-state map of the S1 projection (Alg. 2 with zero
// data: u = K x, x^c = Abar^c x), and the cost-weight gradients.
#include "device_common.h"

#include <algorithm>

namespace spk {

// J_G d on a translated SOC block by one wavefront: vector part of len <=
// 128 entries (lane o holds entries o and o + 64), then the two trailing
// scalars a (entry len) and b (entry len + 1); b_ is the block of b*.
template <typename S>
__device__ void soc_jg_wave(const S* __restrict__ b_, const S* __restrict__ din, S* __restrict__ dout, int len,
                            S al, int lane) {
  const S ia = S(1) / al;
  S bv[2], dv[2];
  double r2p = 0;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int o = lane + 64 * s;
    const int oo = o < len ? o : 0;
    bv[s] = o < len ? b_[oo] : S(0);
    dv[s] = o < len ? din[oo] : S(0);
    r2p += (double)(bv[s] * ia) * (double)(bv[s] * ia);
  }
  const S va = b_[len] * ia - S(0.5);
  const S t = b_[len + 1] * ia + S(0.5);
  const double r2 = team_sum<64>(r2p) + (double)va * (double)va;
  const S r = (S)sqrt(r2);
  const S da = din[len], dt = din[len + 1];
  if (r <= t) {  // inside the cone: proj Jacobian = I, J_G = 0
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (lane + 64 * s < len) dout[lane + 64 * s] = S(0);
    if (lane == 0) {
      dout[len] = S(0);
      dout[len + 1] = S(0);
    }
    return;
  }
  if (r <= -t) {  // polar cone: proj Jacobian = 0, J_G = I
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (lane + 64 * s < len) dout[lane + 64 * s] = dv[s];
    if (lane == 0) {
      dout[len] = da;
      dout[len + 1] = dt;
    }
    return;
  }
  // J_proj (x, t) -> 1/2 [ (1 + t/r) dx - (t/r) xh (xh.dx) + xh dt ; xh.dx + dt ],
  // xh = x / r, x = (b_vec / alpha, b_a / alpha - 1/2)
  const S ir = S(1) / r;
  double xdp = 0;
#pragma unroll
  for (int s = 0; s < 2; ++s) xdp += (double)(bv[s] * ia * ir) * (double)dv[s];
  const double xd = team_sum<64>(xdp) + (double)(va * ir) * (double)da;
  const S tr = t * ir;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    if (lane + 64 * s < len) {
      const S xh = bv[s] * ia * ir;
      const S jp = S(0.5) * ((S(1) + tr) * dv[s] - tr * xh * (S)xd + xh * dt);
      dout[lane + 64 * s] = dv[s] - jp;
    }
  }
  if (lane == 0) {
    const S xh = va * ir;
    const S jp = S(0.5) * ((S(1) + tr) * da - tr * xh * (S)xd + xh * dt);
    dout[len] = da - jp;
    dout[len + 1] = dt - S(0.5) * ((S)xd + dt);
  }
}

// out = J_G(b*) w on every block of S3: one wavefront per family (group 1
// of i, group 2 of each child, group 3 of leaf children), grid-stride.
template <typename S>
__global__ void __launch_bounds__(256) k_jg(DevProb<S> P, const S* __restrict__ b, const S* __restrict__ w,
                                            S* __restrict__ out, long long is) {
  b += (size_t)blockIdx.y * is;  // instance blockIdx.y of a batch (stride is)
  w += (size_t)blockIdx.y * is;
  out += (size_t)blockIdx.y * is;
  const int lane = threadIdx.x & 63;
  const Off<S> O(P);
  const int nx = P.nx, nu = P.nu;
  const S al = P.alpha, ia = S(1) / al;
  for (int i = blockIdx.x * 4 + (int)(threadIdx.x >> 6); i < P.nl; i += gridDim.x * 4) {
    const int fc = P.fc[i], n = P.nch[i];
    const long long e1 = O.e1(i);
    for (int k = lane; k < 2 * n; k += 64) out[e1 + k] = (b[e1 + k] <= S(0)) ? w[e1 + k] : S(0);  // K*: max(.,0)
    if (lane == 0) {
      out[e1 + 2 * n] = S(0);                                                       // free entry
      out[e1 + 2 * n + 1] = (b[e1 + 2 * n + 1] <= S(0)) ? w[e1 + 2 * n + 1] : S(0);  // R_+
    }
    for (int o = lane; o < nx; o += 64) {
      const long long e = O.e1x(i) + o;
      const S v = b[e] * ia;
      const bool in = v > P.xlo[(size_t)i * nx + o] && v < P.xhi[(size_t)i * nx + o];
      out[e] = in ? S(0) : w[e];
    }
    for (int o = lane; o < nu; o += 64) {
      const long long e = O.e1u(i) + o;
      const S v = b[e] * ia;
      const bool in = v > P.ulo[(size_t)i * nu + o] && v < P.uhi[(size_t)i * nu + o];
      out[e] = in ? S(0) : w[e];
    }
    for (int c = fc; c < fc + n; ++c) {
      const long long e2 = O.e2(c);
      soc_jg_wave<S>(b + e2, w + e2, out + e2, nx + nu, al, lane);
      if (c >= P.nl) {
        const long long e3 = O.e3(c);
        for (int o = lane; o < nx; o += 64) {
          const S v = b[e3 + o] * ia;
          const bool in = v > P.xlo[(size_t)c * nx + o] && v < P.xhi[(size_t)c * nx + o];
          out[e3 + o] = in ? S(0) : w[e3 + o];
        }
        soc_jg_wave<S>(b + e3 + nx, w + e3 + nx, out + e3 + nx, nx, al, lane);
      }
    }
  }
}

// Inputs of the adjoint of every instance in one launch: v* (and the root
// state) gathered from the callers' buffers, the cotangent g = gV on s^0 and
// gu0 on u^0 (element u0off on), and w = g. Instance b sits `is` elements
// apart; tab holds the pointers of the instances (v*, x0, gu0 or null). A
// launch bound, not a bandwidth bound: 64 instances of the 95-node tree took
// 4 copies each (and a synchronisation for gu0).
template <typename S>
__global__ void __launch_bounds__(256) k_adj_load(long long nv, int nx, int nu, long long u0off, double gV,
                                                  const AdjPtrs<S>* __restrict__ tab, long long is,
                                                  S* __restrict__ v, double* __restrict__ x0s, S* __restrict__ g,
                                                  S* __restrict__ w) {
  const AdjPtrs<S> t = tab[blockIdx.y];
  const size_t o = (size_t)blockIdx.y * is;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < nv; e += (long long)gridDim.x * blockDim.x) {
    if (v) v[o + e] = t.vstar[e];
    S c = S(0);
    if (e == 0) c = (S)gV;
    else if (t.gu0 && e >= u0off && e < u0off + nu) c = (S)t.gu0[e - u0off];
    g[o + e] = c;
    w[o + e] = c;
    if (x0s && e < nx) x0s[(size_t)blockIdx.y * nx + e] = t.x0[e];
  }
}

// J_G d on a translated SOC block held in registers (soc_jg_wave's formulas):
// vector part bv, dv in two components per lane (zero past the end), the
// scalars ba, bb of b* and da, dt of d in every lane; results in place of dv,
// da, dt.
template <typename S>
__device__ __forceinline__ void soc_jg_regs(const S (&bv)[2], S (&dv)[2], S ba, S bb, S& da, S& dt, S al) {
  const S ia = S(1) / al;
  double r2p = 0;
#pragma unroll
  for (int s = 0; s < 2; ++s) r2p += (double)(bv[s] * ia) * (double)(bv[s] * ia);
  const S va = ba * ia - S(0.5);
  const S t = bb * ia + S(0.5);
  const S r = (S)sqrt(team_sum<64>(r2p) + (double)va * (double)va);
  if (r <= t) {  // inside the cone: J_G = 0
    dv[0] = dv[1] = da = dt = S(0);
    return;
  }
  if (r <= -t) return;  // polar cone: J_G = I
  const S ir = S(1) / r;
  double xdp = 0;
#pragma unroll
  for (int s = 0; s < 2; ++s) xdp += (double)(bv[s] * ia * ir) * (double)dv[s];
  const double xd = team_sum<64>(xdp) + (double)(va * ir) * (double)da;
  const S tr = t * ir;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const S xh = bv[s] * ia * ir;
    dv[s] -= S(0.5) * ((S(1) + tr) * dv[s] - tr * xh * (S)xd + xh * dt);
  }
  const S xh = va * ir;
  const S ja = S(0.5) * ((S(1) + tr) * da - tr * xh * (S)xd + xh * dt);
  const S jt = S(0.5) * ((S)xd + dt);
  da -= ja;
  dt -= jt;
}

// First half of an application of the transposed operator, up to the sweeps:
//   lb = J_G(b*) w_eta,  tz = L* lb,  cz = w_z + 2 alpha tz,
// then the pre-pass of J_f cz (zero dual part): xbar, ubar = cz on (x, u), q =
// -cz_x at leaves, the S2 projection of the (y, tau, s) blocks into la, and
// la's s^0 = cz's (the identity there). One wavefront per family and instance:
// every row of lb and column of tz it needs is its own, but for s of a nonleaf
// child, whose one row (the child's s-row) it computes again. One launch in
// place of five (J_G, L*, the combination, the pre-pass, the s^0 copy), which
// took 26 us per application on the 95-node tree in FP64. n <= 64 children. The
// combination is formed in FP64 with the unrounded alpha and rounded once.
// Arrays of instance b: w at + b ws, the others at + b is.
template <typename S>
__global__ void __launch_bounds__(256) k_adj_front(DevProb<S> P, const long long* __restrict__ spos,
                                                   const S* __restrict__ bs, const S* __restrict__ w, long long ws,
                                                   S* __restrict__ lb, S* __restrict__ tz, S* __restrict__ cz,
                                                   S* __restrict__ la, S* __restrict__ xbar, S* __restrict__ ubar,
                                                   S* __restrict__ q, long long is, int tiles, double alpha2) {
  const size_t inst = blockIdx.y;
  const int nx = P.nx, nu = P.nu, K = nx + nu;
  bs += inst * is;
  const S* wz = w + inst * ws;
  const S* we = wz + P.nz;
  lb += inst * is;
  tz += inst * is;
  cz += inst * is;
  la += inst * is;
  const size_t cs = tiles ? kTileCols : 1;  // from one entry to the next
  const size_t bx = tiles ? tile_base(inst, (size_t)P.nn * nx) : inst * (size_t)P.nn * nx;
  xbar += bx;
  q += bx;
  ubar += tiles ? tile_base(inst, (size_t)P.nn * nu) : inst * (size_t)P.nn * nu;
  const int lane = threadIdx.x & 63;
  const Off<S> O(P);
  const S al = P.alpha, ia = S(1) / al;
  const int i = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (i >= P.nl) return;
  const int fc = P.fc[i], n = P.nch[i];
  const long long e1 = O.e1(i), e1s = e1 + 2LL * n + 1, zb = O.z2(i);
  const bool leaf = fc >= P.nl;
  // (an FP64 problem's alpha is the unrounded one: no argument held for it)
  const double al2 = sizeof(S) == 8 ? 2.0 * (double)al : alpha2;
  auto comb = [&](long long e, S t) { return (S)((double)wz[e] + al2 * (double)t); };
  auto put = [&](long long e, S t) {  // one column: tz, cz; returns cz
    const S c = comb(e, t);
    tz[e] = t;
    cz[e] = c;
    return c;
  };
  // ---- group 1: the s-row and the y rows (lane k: y1, y2 of child k)
  const S res = bs[e1s] <= S(0) ? we[e1s] : S(0);
  S y1 = 0, y2 = 0, th = 0, sh = 0;
  if (lane < n) {
    const S l1 = bs[e1 + lane] <= S(0) ? we[e1 + lane] : S(0);
    const S l2 = bs[e1 + n + lane] <= S(0) ? we[e1 + n + lane] : S(0);
    lb[e1 + lane] = l1;
    lb[e1 + n + lane] = l2;
    y1 = put(zb + lane, l1 - P.p[fc + lane] * res);
    y2 = put(zb + n + lane, l2);
    if (!leaf) {  // s of child `lane`: its s-row, owned (and stored) by that child's family
      const long long ec = O.e1s(fc + lane);
      sh = comb(zb + 3LL * n + 1 + lane, bs[ec] <= S(0) ? we[ec] : S(0));
    }
  }
  const S y3 = comb(zb + 2 * n, S(0) - res);
  if (lane == 0) {
    lb[e1 + 2 * n] = S(0);  // the free entry
    lb[e1s] = res;
    put(zb + 2 * n, S(0) - res);
    const S c = put(spos[i], res);
    if (i == 0) la[0] = c;
  }
  // ---- the box rows (x, u) of group 1 and the columns x^i, u^i
  bool on[2];
  S acc[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int k = lane + 64 * s;
    on[s] = k < K;
    acc[s] = 0;
    if (!on[s]) continue;
    const long long e = e1s + 1 + k;
    const size_t bi = k < nx ? (size_t)i * nx + k : (size_t)i * nu + (k - nx);
    const S v = bs[e] * ia;
    const bool in = v > (k < nx ? P.xlo : P.ulo)[bi] && v < (k < nx ? P.xhi : P.uhi)[bi];
    acc[s] = in ? S(0) : we[e];
    lb[e] = acc[s];
  }
  // ---- group 2 of every child, group 3 of leaf children
  for (int c = fc; c < fc + n; ++c) {
    const long long e2 = O.e2(c);
    S bv[2], dv[2], sc[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int k = lane + 64 * s;
      bv[s] = on[s] ? bs[e2 + k] : S(0);
      dv[s] = on[s] ? we[e2 + k] : S(0);
      sc[s] = !on[s] ? S(0) : (k < nx ? P.sq[(size_t)c * nx + k] : P.sr[(size_t)c * nu + (k - nx)]);
    }
    S da = we[e2 + K], dt = we[e2 + K + 1];
    soc_jg_regs<S>(bv, dv, bs[e2 + K], bs[e2 + K + 1], da, dt, al);
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (on[s]) {
        lb[e2 + lane + 64 * s] = dv[s];
        acc[s] += sc[s] * dv[s];
      }
    if (lane == 0) {
      lb[e2 + K] = da;
      lb[e2 + K + 1] = dt;
    }
    if (lane == c - fc) th = put(zb + 2LL * n + 1 + (c - fc), S(0.5) * (da + dt));
    if (!leaf) continue;
    const long long e3 = O.e3(c);
    const bool ox = lane < nx;
    S lx = 0, sq = 0;
    S b3[2] = {S(0), S(0)}, d3[2] = {S(0), S(0)};
    if (ox) {
      const S v = bs[e3 + lane] * ia;
      const size_t bi = (size_t)c * nx + lane;
      lx = v > P.xlo[bi] && v < P.xhi[bi] ? S(0) : we[e3 + lane];
      sq = P.sqN[bi];
      b3[0] = bs[e3 + nx + lane];
      d3[0] = we[e3 + nx + lane];
    }
    S ea = we[e3 + 2 * nx], eb = we[e3 + 2 * nx + 1];
    soc_jg_regs<S>(b3, d3, bs[e3 + 2 * nx], bs[e3 + 2 * nx + 1], ea, eb, al);
    if (ox) {
      lb[e3 + lane] = lx;
      lb[e3 + nx + lane] = d3[0];
      q[((size_t)c * nx + lane) * cs] = -put(O.x(c) + lane, lx + sq * d3[0]);
    }
    if (lane == 0) {
      lb[e3 + 2 * nx] = ea;
      lb[e3 + 2 * nx + 1] = eb;
    }
    if (lane == c - fc) sh = put(zb + 3LL * n + 1 + (c - fc), S(0.5) * (ea + eb));
  }
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int k = lane + 64 * s;
    if (!on[s]) continue;
    if (k < nx) xbar[((size_t)i * nx + k) * cs] = put(O.x(i) + k, acc[s]);
    else ubar[((size_t)i * nu + (k - nx)) * cs] = put(O.u(i) + (k - nx), acc[s]);
  }
  // ---- S2 projection of the (y, tau, s) block (closed form, as the pre-pass)
  const S a = P.a[i], cc = a * a + S(3);
  const S g = a * y1 - y2 + y3 - th - sh;
  const S corr = (S)team_sum<64>(lane < n ? (double)g : 0.0) / (cc + S(n));
  const S pr = (g - corr) / cc;
  const S Ws = (S)team_sum<64>(lane < n ? (double)pr : 0.0);
  if (lane < n) {
    la[zb + lane] = y1 - a * pr;
    la[zb + n + lane] = y2 + pr;
    la[zb + 2LL * n + 1 + lane] = th + pr;
    la[zb + 3LL * n + 1 + lane] = sh + pr;
  }
  if (lane == 0) la[zb + 2 * n] = y3 - Ws;
}

// Second half: out = a v + s (J_T' w) + c g with J_T' w = (la - alpha tz, lb -
// alpha L la): A(w) = J_T' w + g with (a, s, c) = (0, 1, 1), the next Krylov
// vector v - J_T' v (the cotangent cancels) with (1, -1, 0). Wavefronts run
// over the z entries first, then a family (or more) each for the rows of L la.
// One launch in place of four (L, three combinations); al is the unrounded
// alpha. Bound by the latency of its loads.
template <typename S>
__global__ void __launch_bounds__(256) k_adj_back(DevProb<S> P, double al, double a, const S* __restrict__ v, long long vs,
                                                  double sg, const S* __restrict__ la, const S* __restrict__ tz,
                                                  const S* __restrict__ lb, double cg, const S* __restrict__ g,
                                                  S* __restrict__ out, long long os, long long is) {
  const size_t inst = blockIdx.y;
  v += inst * vs;
  out += inst * os;
  la += inst * is;
  tz += inst * is;
  lb += inst * is;
  g += inst * is;
  const int lane = threadIdx.x & 63;
  const Off<S> O(P);
  const int nx = P.nx, nu = P.nu, K = nx + nu;
  auto put = [&](long long e, double j) {
    double r = sg * j;
    if (a != 0.0) r += a * (double)v[e];
    if (cg != 0.0) r += cg * (double)g[e];
    out[e] = (S)r;
  };
  for (long long e = blockIdx.x * 256LL + threadIdx.x; e < P.nz; e += gridDim.x * 256LL)
    put(e, (double)la[e] - al * (double)tz[e]);
  const long long nz = P.nz;
  auto row = [&](long long e, S Ll) { put(nz + e, (double)lb[e] - al * (double)Ll); };
  for (int i = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); i < P.nl; i += gridDim.x * 4) {
    const int fc = P.fc[i], n = P.nch[i];
    const long long zb = O.z2(i), e1 = O.e1(i), e1x = e1 + 2LL * n + 2;
    double by = 0;
    for (int k = lane; k < 2 * n + 1; k += 64) {
      const S y = la[zb + k];
      row(e1 + k, y);
      if (k < n) by += (double)(P.p[fc + k] * y);
    }
    by = team_sum<64>(by) + (double)la[zb + 2 * n];
    if (lane == 0) row(e1 + 2 * n + 1, la[O.s(i)] - (S)by);
    S xu[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int k = lane + 64 * s;
      xu[s] = k < K ? la[k < nx ? O.x(i) + k : O.u(i) + (k - nx)] : S(0);
      if (k < K) row(e1x + k, xu[s]);
    }
    for (int c = fc; c < fc + n; ++c) {
      const long long e2 = O.e2(c);
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        const int k = lane + 64 * s;
        if (k < K) row(e2 + k, (k < nx ? P.sq[(size_t)c * nx + k] : P.sr[(size_t)c * nu + (k - nx)]) * xu[s]);
      }
      if (lane < 2) row(e2 + K + lane, S(0.5) * la[zb + 2LL * n + 1 + (c - fc)]);
      if (c >= P.nl) {
        const long long e3 = O.e3(c);
        if (lane < nx) {
          const S xc = la[O.x(c) + lane];
          row(e3 + lane, xc);
          row(e3 + nx + lane, P.sqN[(size_t)c * nx + lane] * xc);
        }
        if (lane < 2) row(e3 + 2 * nx + lane, S(0.5) * la[zb + 3LL * n + 1 + (c - fc)]);
      }
    }
  }
}

// Transpose of the root-state map Phi of the S1 projection, one stage per
// launch (stage N-1 .. 0) for every instance: mu^j = c_x^j at leaves, mu^i =
// c_x^i + K^i' c_u^i + sum_c Abar^c' mu^c; mu^0 is the gradient with respect
// to x0, written to gx0. One wavefront per (node, instance), lane o on
// component o (nx <= 64): the rows of K and Abar are read coalesced and the
// sums run in the order of the formula. Bound by the latency of a stage's
// chain; one thread per node walked nx (nu + n nx) dependent loads (85 us per
// stage on the 95-node tree in FP64, once per instance: 43 of the 60 ms that a
// 64-instance adjoint of 32 applications took; it takes 7.6 ms in all now).
template <typename S>
__global__ void __launch_bounds__(256) k_phiT(DevProb<S> P, const S* __restrict__ cz, long long is,
                                              S* __restrict__ mu, long long ms, int first, int count,
                                              const AdjPtrs<S>* __restrict__ tab) {
  const int lane = threadIdx.x & 63;
  const int f = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (f >= count) return;
  const int i = first + f;
  cz += (size_t)blockIdx.y * is;
  mu += (size_t)blockIdx.y * ms;
  const Off<S> O(P);
  const int nx = P.nx, nu = P.nu, fc = P.fc[i], n = P.nch[i];
  const int o = lane < nx ? lane : 0;
  double acc = (double)cz[O.x(i) + o];
  const S* K = P.KR + (size_t)i * nu * nx + o;
  const S* cu = cz + O.u(i);
#pragma unroll 8
  for (int j = 0; j < nu; ++j) acc += (double)K[(size_t)j * nx] * (double)cu[j];
  for (int c = fc; c < fc + n; ++c) {
    const S* Ab = P.AbR + (size_t)c * nx * nx + o;  // row-major Abar: (Abar' mu)_o = sum_r Abar[r][o] mu_r
    const S* m = c >= P.nl ? cz + O.x(c) : mu + (size_t)c * nx;
#pragma unroll 8
    for (int r = 0; r < nx; ++r) acc += (double)Ab[(size_t)r * nx] * (double)m[r];
  }
  if (lane < nx) {
    mu[(size_t)i * nx + lane] = (S)acc;
    if (i == 0) tab[blockIdx.y].gx0[lane] = (double)(S)acc;
  }
}

// Cost-weight gradients from the adjoint quantities: for a non-root c with
// ancestor i, d/dq^c_k = alpha (x*_{i,k} lb_{c,k} - la_{x^i,k} eta*_{c,k}) / (2 sqrt(q^c_k))
// on the group-2 x rows; for a leaf j, the same with group 3 and Q_N. Every
// entry of both outputs is written (row 0 and the other rows of gqN are
// zero), one thread per entry and instance.
template <typename S>
__global__ void __launch_bounds__(256) k_grad_q(DevProb<S> P, const S* __restrict__ vstar, const S* __restrict__ la,
                                                const S* __restrict__ lb, long long is,
                                                const AdjPtrs<S>* __restrict__ tab) {
  const long long e = blockIdx.x * 256LL + threadIdx.x;
  const int nx = P.nx;
  if (e >= (long long)P.nn * nx) return;
  const AdjPtrs<S> t = tab[blockIdx.y];
  const size_t b = (size_t)blockIdx.y * is;
  const int c = (int)(e / nx), k = (int)(e - (long long)c * nx);
  const Off<S> O(P);
  const S* z = vstar ? vstar + b : t.vstar;
  const S* eta = z + P.nz;
  la += b;
  lb += b;
  const double al = (double)P.alpha;
  if (t.gq) {
    double out = 0.0;
    if (c > 0) {
      const int i = P.anc[c];
      const long long e2 = O.e2(c);
      const double sq = (double)P.sq[(size_t)c * nx + k];
      const double d = al * ((double)z[O.x(i) + k] * (double)lb[e2 + k] - (double)la[O.x(i) + k] * (double)eta[e2 + k]);
      out = d / (2.0 * sq);
    }
    t.gq[e] = out;
  }
  if (t.gqN) {
    double out = 0.0;
    if (c >= P.nl) {
      const long long e3q = O.e3(c) + nx;
      const double sq = (double)P.sqN[(size_t)c * nx + k];
      const double d = al * ((double)z[O.x(c) + k] * (double)lb[e3q + k] - (double)la[O.x(c) + k] * (double)eta[e3q + k]);
      out = sq > 0.0 ? d / (2.0 * sq) : 0.0;
    }
    t.gqN[e] = out;
  }
}

// max |a - b| over n entries, per block, then over blocks (one launch each)
template <typename S>
__global__ void k_maxdiff(long long n, const S* __restrict__ a, const S* __restrict__ b,
                          double* __restrict__ partials) {
  __shared__ double red[256];
  double m = 0;
  for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < n;
       e += (long long)gridDim.x * blockDim.x) {
    m = fmax(m, fabs((double)a[e] - (double)b[e]));
  }
  red[threadIdx.x] = m;
  __syncthreads();
  for (int s = blockDim.x / 2; s >= 1; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) partials[blockIdx.x] = red[0];
}
__global__ void k_max_final(const double* __restrict__ partials, int nblk, double* __restrict__ out) {
  if (threadIdx.x != 0) return;
  double m = 0;
  for (int b = 0; b < nblk; ++b) m = fmax(m, partials[b]);
  out[0] = m;
}

template <typename S>
__global__ void k_copy_elem(S* dst, const S* src) { dst[0] = src[0]; }

// ---- launchers
template <typename S>
hipError_t launch_copy_elem(S* dst, const S* src, hipStream_t st) {
  hipLaunchKernelGGL(k_copy_elem<S>, dim3(1), dim3(1), 0, st, dst, src);
  return hipGetLastError();
}
template <typename S>
hipError_t launch_jg(const Problem& P, const S* b, const S* w, S* out, hipStream_t st) {
  const DevProb<S>& D = (sizeof(S) == 8) ? *reinterpret_cast<const DevProb<S>*>(&P.dp64)
                                         : *reinterpret_cast<const DevProb<S>*>(&P.dp32);
  hipLaunchKernelGGL(k_jg<S>, dim3(family_wave_blocks(P.tree->nl)), dim3(256), 0, st, D, b, w, out, 0LL);
  return hipGetLastError();
}
template <typename S>
hipError_t launch_jg_batch(const Problem& P, const S* b, const S* w, S* out, long long is, int B, hipStream_t st) {
  const DevProb<S>& D = (sizeof(S) == 8) ? *reinterpret_cast<const DevProb<S>*>(&P.dp64)
                                         : *reinterpret_cast<const DevProb<S>*>(&P.dp32);
  hipLaunchKernelGGL(k_jg<S>, dim3(family_wave_blocks(P.tree->nl), B), dim3(256), 0, st, D, b, w, out, is);
  return hipGetLastError();
}
template <typename S>
hipError_t launch_adj_load(const Problem& P, double gV, const AdjPtrs<S>* tab, long long is, int B, S* v, double* x0s,
                           S* g, S* w, hipStream_t st) {
  const long long nv = P.nz + P.neta;
  const int nb = (int)std::min<long long>((nv + 255) / 256, 64);
  hipLaunchKernelGGL(k_adj_load<S>, dim3(nb, B), dim3(256), 0, st, nv, P.nx, P.nu,
                     1 + (long long)P.tree->nn * P.nx, gV, tab, is, v, x0s, g, w);
  return hipGetLastError();
}
template <typename S>
hipError_t launch_adj_front(const Problem& P, const S* bs, const S* w, long long ws, S* lb, S* tz, S* cz, S* la,
                            S* xbar, S* ubar, S* q, long long is, int B, bool tiles, hipStream_t st) {
  const DevProb<S>& D = (sizeof(S) == 8) ? *reinterpret_cast<const DevProb<S>*>(&P.dp64)
                                         : *reinterpret_cast<const DevProb<S>*>(&P.dp32);
  hipLaunchKernelGGL(k_adj_front<S>, dim3((P.tree->nl + 3) / 4, B), dim3(256), 0, st, D, P.d_spos, bs, w, ws, lb, tz,
                     cz, la, xbar, ubar, q, is, tiles ? 1 : 0, 2.0 * P.alpha);
  return hipGetLastError();
}
template <typename S>
hipError_t launch_adj_back(const Problem& P, double a, const S* v, long long vs, double sg, const S* la, const S* tz,
                           const S* lb, double cg, const S* g, S* out, long long os, long long is, int B,
                           hipStream_t st) {
  const DevProb<S>& D = (sizeof(S) == 8) ? *reinterpret_cast<const DevProb<S>*>(&P.dp64)
                                         : *reinterpret_cast<const DevProb<S>*>(&P.dp32);
  hipLaunchKernelGGL(k_adj_back<S>, dim3(family_wave_blocks(P.tree->nl), B), dim3(256), 0, st, D, P.alpha, a, v, vs, sg,
                     la, tz, lb, cg, g, out, os, is);
  return hipGetLastError();
}
template <typename S>
hipError_t launch_phiT(const Problem& P, const S* cz, long long is, S* mu, long long ms, int B,
                       const AdjPtrs<S>* tab, hipStream_t st) {
  const DevProb<S>& D = (sizeof(S) == 8) ? *reinterpret_cast<const DevProb<S>*>(&P.dp64)
                                         : *reinterpret_cast<const DevProb<S>*>(&P.dp32);
  const Tree& T = *P.tree;
  for (int t = T.N - 1; t >= 0; --t) {
    const int first = T.stage_off[t], count = T.stage_off[t + 1] - first;
    hipLaunchKernelGGL(k_phiT<S>, dim3((count + 3) / 4, B), dim3(256), 0, st, D, cz, is, mu, ms, first, count, tab);
  }
  return hipGetLastError();
}
template <typename S>
hipError_t launch_grad_q(const Problem& P, const S* vstar, const S* la, const S* lb, long long is, int B,
                         const AdjPtrs<S>* tab, hipStream_t st) {
  const DevProb<S>& D = (sizeof(S) == 8) ? *reinterpret_cast<const DevProb<S>*>(&P.dp64)
                                         : *reinterpret_cast<const DevProb<S>*>(&P.dp32);
  const long long ne = (long long)P.tree->nn * P.nx;
  hipLaunchKernelGGL(k_grad_q<S>, dim3((unsigned)((ne + 255) / 256), B), dim3(256), 0, st, D, vstar, la, lb, is, tab);
  return hipGetLastError();
}
template <typename S>
hipError_t launch_maxdiff(long long n, const S* a, const S* b, double* partials, double* out, hipStream_t st) {
  const int nb = dots_blocks(n);
  hipLaunchKernelGGL(k_maxdiff<S>, dim3(nb), dim3(256), 0, st, n, a, b, partials);
  hipLaunchKernelGGL(k_max_final, dim3(1), dim3(64), 0, st, partials, nb, out);
  return hipGetLastError();
}

#define SPK_BINST(S)                                                                                  \
  template hipError_t launch_adj_front<S>(const Problem&, const S*, const S*, long long, S*, S*, S*, S*, S*, S*, S*, \
                                          long long, int, bool, hipStream_t);                         \
  template hipError_t launch_adj_back<S>(const Problem&, double, const S*, long long, double, const S*, const S*,    \
                                         const S*, double, const S*, S*, long long, long long, int, hipStream_t);    \
  template hipError_t launch_copy_elem<S>(S*, const S*, hipStream_t);                                 \
  template hipError_t launch_jg<S>(const Problem&, const S*, const S*, S*, hipStream_t);              \
  template hipError_t launch_jg_batch<S>(const Problem&, const S*, const S*, S*, long long, int, hipStream_t); \
  template hipError_t launch_adj_load<S>(const Problem&, double, const AdjPtrs<S>*, long long, int, S*, double*, S*, \
                                         S*, hipStream_t);                                            \
  template hipError_t launch_phiT<S>(const Problem&, const S*, long long, S*, long long, int,         \
                                     const AdjPtrs<S>*, hipStream_t);                                 \
  template hipError_t launch_grad_q<S>(const Problem&, const S*, const S*, const S*, long long, int,  \
                                       const AdjPtrs<S>*, hipStream_t);                               \
  template hipError_t launch_maxdiff<S>(long long, const S*, const S*, double*, double*, hipStream_t);
SPK_BINST(double)
SPK_BINST(float)

}  // namespace spk
