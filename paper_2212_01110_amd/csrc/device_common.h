// Device code shared by the per-stage kernels and the batched block engine:
// canonical offsets, team reductions, proximal maps and the per-family steps
// of the CP operator (section 5 splitting; Alg. 2 sweeps).
#pragma once
#include "spock_internal.h"

#include <math.h>

namespace spk {

// ---------------------------------------------------------------- helpers
__device__ __forceinline__ void wave_lds_sync() {
  // Teams live inside one wavefront and exchange values through LDS only:
  // the ordering is at wavefront scope and for LDS alone, so global loads
  // stay free to move across it.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// The value of the partner lane of a butterfly step of 2^k lanes, the steps
// taken from the widest down: 32 and 16 (and 4 in a team of 8) by shuffles, 8
// to 1 by rotations of a 16-lane row. A rotation by M reaches a lane whose
// value equals that of lane ^ M once the wider steps have made the row periodic
// in 2 M. A shuffle through LDS costs about 120 cycles a step, a rotation a
// few.
template <int M, int T>
__device__ __forceinline__ double lane_partner(double v) {
  unsigned w[2];
  __builtin_memcpy(w, &v, 8);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if constexpr (M <= 2) w[k] = (unsigned)__builtin_amdgcn_update_dpp((int)w[k], (int)w[k], M == 1 ? 0xB1 : 0x4E, 0xF, 0xF, false);
    else if constexpr (M <= 8 && T >= 16) w[k] = (unsigned)__builtin_amdgcn_update_dpp((int)w[k], (int)w[k], 0x120 + M, 0xF, 0xF, false);
    else w[k] = (unsigned)__shfl_xor((int)w[k], M, 64);
  }
  double o;
  __builtin_memcpy(&o, w, 8);
  return o;
}
// Sum (maximum) over the team of T lanes, the same bits in every lane.
template <int T>
__device__ __forceinline__ double team_sum(double v) {
  if constexpr (T >= 64) v += lane_partner<32, T>(v);
  if constexpr (T >= 32) v += lane_partner<16, T>(v);
  if constexpr (T >= 16) v += lane_partner<8, T>(v);
  if constexpr (T >= 8) v += lane_partner<4, T>(v);
  if constexpr (T >= 4) v += lane_partner<2, T>(v);
  if constexpr (T >= 2) v += lane_partner<1, T>(v);
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, lane_partner<32, 64>(v));
  v = fmax(v, lane_partner<16, 64>(v));
  v = fmax(v, lane_partner<8, 64>(v));
  v = fmax(v, lane_partner<4, 64>(v));
  v = fmax(v, lane_partner<2, 64>(v));
  return fmax(v, lane_partner<1, 64>(v));
}

template <typename S>
__device__ __forceinline__ S clampv(S v, S lo, S hi) {
  return v < lo ? lo : (v > hi ? hi : v);
}

// acc[c] += sum_k Mt[k*nout + o] * vin[k], o = lane + c*T (o < nout);
// D bounds the output dimension (compile-time chunk count C = ceil(D / T)).
template <typename S, int T, int D = kMaxDim>
__device__ __forceinline__ void mv_acc(S (&acc)[(D + T - 1) / T], const S* __restrict__ Mt,
                                       int nin, int nout, const S* vin, int lane) {
  constexpr int C = (D + T - 1) / T;
  int k = 0;
  for (; k + 4 <= nin; k += 4) {
    const S v0 = vin[k], v1 = vin[k + 1], v2 = vin[k + 2], v3 = vin[k + 3];
    const S* r0 = Mt + (size_t)k * nout;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int o = lane + c * T;
      if (o < nout) {
        const S m0 = r0[o], m1 = r0[nout + o], m2 = r0[2 * nout + o], m3 = r0[3 * nout + o];
        acc[c] += m0 * v0 + m1 * v1 + m2 * v2 + m3 * v3;
      }
    }
  }
  for (; k < nin; ++k) {
    const S vk = vin[k];
    const S* r0 = Mt + (size_t)k * nout;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int o = lane + c * T;
      if (o < nout) acc[c] += r0[o] * vk;
    }
  }
}

// Element i of an array. IX = unsigned: the byte offset fits 32 bits (the
// caller's rule), so that a divergent index costs one multiply-add on a uniform
// base; IX = long long: any size.
template <typename S, typename IX>
__device__ __forceinline__ const S& at(const S* p, IX i) {
  if constexpr (sizeof(IX) == 4) return *reinterpret_cast<const S*>(reinterpret_cast<const char*>(p) + (unsigned)(i * (IX)sizeof(S)));
  else return p[i];
}
template <typename S, typename IX>
__device__ __forceinline__ S& at(S* p, IX i) {
  if constexpr (sizeof(IX) == 4) return *reinterpret_cast<S*>(reinterpret_cast<char*>(p) + (unsigned)(i * (IX)sizeof(S)));
  else return p[i];
}

// The array (a for states, b for inputs) that a lane reads at i: with 32-bit
// offsets both through the base a, i moved by the arrays' distance (they sit
// in one allocation, b above a), so that the base stays uniform.
template <typename S, typename IX>
__device__ __forceinline__ const S* pair_base(const S* a, const S* b, bool first, IX& i) {
  if constexpr (sizeof(IX) == 4) {
    i += first ? IX(0) : (IX)(b - a);
    return a;
  } else {
    return first ? a : b;
  }
}

// Offsets in the canonical layout (closed forms of the breadth-first sizes).
template <typename S, typename IX = long long>
struct Off {
  const DevProb<S>& P;
  __device__ Off(const DevProb<S>& p) : P(p) {}
  __device__ IX x(int i) const { return 1 + (IX)i * P.nx; }
  __device__ IX u(int i) const { return (IX)P.zU + (IX)i * P.nu; }
  // z2 block of nonleaf i: y (2n+1), tau (n), s (n)
  __device__ IX z2(int i) const { return (IX)P.zZ2 + (IX)4 * (P.fc[i] - 1) + i; }
  // slot of s^c in its ancestor's block (s^0 at 0)
  __device__ IX s(int c) const {
    if (c == 0) return 0;
    const int a = P.anc[c];
    const int n = P.nch[a];
    return z2(a) + 3 * n + 1 + (c - P.fc[a]);
  }
  __device__ IX tau(int c) const {
    const int a = P.anc[c];
    const int n = P.nch[a];
    return z2(a) + 2 * n + 1 + (c - P.fc[a]);
  }
  // eta group 1 of nonleaf i: y (2n+1), s-row, x (nx), u (nu)
  __device__ IX e1(int i) const {
    return (IX)2 * (P.fc[i] - 1) + (IX)i * (2 + P.nx + P.nu);
  }
  __device__ IX e1s(int i) const { return e1(i) + (IX)2 * P.nch[i] + 1; }
  __device__ IX e1x(int i) const { return e1s(i) + 1; }
  __device__ IX e1u(int i) const { return e1x(i) + P.nx; }
  // eta group 2 of non-root c: x (nx), u (nu), a, b
  __device__ IX e2(int c) const { return (IX)P.eE2 + (IX)(c - 1) * (P.nx + P.nu + 2); }
  // eta group 3 of leaf j: x (nx), Q_N^{1/2} x (nx), a, b
  __device__ IX e3(int j) const { return (IX)P.eE3 + (IX)(j - P.nl) * (2 * P.nx + 2); }
};

// Running residual statistics of one lane (FP64).
struct StatAcc {
  double rz2 = 0, re2 = 0, cross = 0, xip = 0, xid = 0;
  __device__ void col(double rz, double Ltre, double ia) {
    rz2 += rz * rz;
    xip = fmax(xip, fabs(rz * ia - Ltre));
  }
  __device__ void row(double re, double Lrz, double ia) {
    re2 += re * re;
    cross += re * Lrz;
    xid = fmax(xid, fabs(re * ia - Lrz));
  }
};

// prox of g* on a translated SOC block (eq. S3-def, shift (0,..,0,1/2,-1/2)):
// out = w - alpha (shift + proj_SOC(w/alpha - shift)). The vector part is
// distributed over the team (wv[c] for components o = lane + c*T < len);
// the two trailing scalars (wa, wb) are held by every lane.
template <typename S, int T, int D = kMaxDim>
__device__ __forceinline__ void soc_prox(const S* wv, S* outv, int len, S wa, S wb, S& outa,
                                         S& outb, S al, int lane) {
  constexpr int C = (D * 2 + T - 1) / T;
  const S ia = S(1) / al;
  double part = 0;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    if (o < len) {
      const double t = (double)(wv[c] * ia);
      part += t * t;
    }
  }
  const S va = wa * ia - S(0.5);
  const S t = wb * ia + S(0.5);
  const double n2 = team_sum<T>(part) + (double)va * (double)va;
  const S nrm = (S)sqrt(n2);
  S scale, pt;
  if (nrm <= t) {
    scale = S(1);
    pt = t;
  } else if (nrm <= -t) {
    scale = S(0);
    pt = S(0);
  } else {
    const S cc = S(0.5) * (nrm + t);
    scale = cc / nrm;
    pt = cc;
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    if (o < len) outv[c] = wv[c] - al * (scale * (wv[c] * ia));
  }
  outa = wa - al * (S(0.5) + scale * va);
  outb = wb - al * (S(-0.5) + pt);
}

// prox of g* on a translated SOC block (eq. S3-def, shift (0,..,0,1/2,-1/2))
// by one wavefront: the vector part in two components per lane (w0 counts if
// on0, w1 if on1), the two trailing scalars in every lane; out = w - alpha
// (shift + proj_SOC(w / alpha - shift)).
template <typename S>
__device__ __forceinline__ void soc_prox_wave(S& w0, bool on0, S& w1, bool on1, S& wa, S& wb, S al) {
  const S ia = S(1) / al;
  const S t0 = w0 * ia, t1 = w1 * ia;
  double part = 0;
  if (on0) part += (double)t0 * (double)t0;
  if (on1) part += (double)t1 * (double)t1;
  const S va = wa * ia - S(0.5);
  const S t = wb * ia + S(0.5);
  const S nrm = (S)sqrt(team_sum<64>(part) + (double)va * (double)va);
  S scale, pt;
  if (nrm <= t) {
    scale = S(1);
    pt = t;
  } else if (nrm <= -t) {
    scale = S(0);
    pt = S(0);
  } else {
    const S cc = S(0.5) * (nrm + t);
    scale = cc / nrm;
    pt = cc;
  }
  w0 = w0 - al * (scale * t0);
  w1 = w1 - al * (scale * t1);
  wa = wa - al * (S(0.5) + scale * va);
  wb = wb - al * (S(-0.5) + pt);
}

// ---------------------------------------------------------------- family pieces
// The functions below run on one team of T lanes (T <= 64, inside one
// wavefront); lane o owns components o, o+T, ... of node vectors.

// xbar, ubar of nonleaf i: (x, u) - alpha (L* eta) on columns x^i, u^i.
template <typename S, int T, int D = kMaxDim>
__device__ __forceinline__ void fam_xbar_ubar(const DevProb<S>& P, const Off<S>& O,
                                              const S* __restrict__ z, const S* __restrict__ eta,
                                              int i, int lane, S (&xb)[(D + T - 1) / T],
                                              S (&ub)[(D + T - 1) / T]) {
  constexpr int C = (D + T - 1) / T;
  const int nx = P.nx, nu = P.nu, fc = P.fc[i], n = P.nch[i];
  const S al = P.alpha;
  const long long e1x = O.e1x(i), e1u = O.e1u(i);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    xb[c] = 0;
    ub[c] = 0;
    if (o < nx) {
      S acc = eta[e1x + o];
      for (int k = 0; k < n; ++k) acc += P.sq[(size_t)(fc + k) * nx + o] * eta[O.e2(fc + k) + o];
      xb[c] = z[O.x(i) + o] - al * acc;
    }
    if (o < nu) {
      S acc = eta[e1u + o];
      for (int k = 0; k < n; ++k) acc += P.sr[(size_t)(fc + k) * nu + o] * eta[O.e2(fc + k) + nx + o];
      ub[c] = z[O.u(i) + o] - al * acc;
    }
  }
}

// q of a child for the backward sweep: -xbar at a leaf (Alg. 2 start), the
// stored q otherwise. Component o < nx.
template <typename S>
__device__ __forceinline__ S fam_child_q(const DevProb<S>& P, const Off<S>& O, const S* __restrict__ z,
                                         const S* __restrict__ eta, const S* __restrict__ qbuf, int ch,
                                         int o) {
  const int nx = P.nx;
  if (ch >= P.nl) {
    const long long e3 = O.e3(ch);
    return -(z[O.x(ch) + o] - P.alpha * (eta[e3 + o] + P.sqN[(size_t)ch * nx + o] * eta[e3 + nx + o]));
  }
  return qbuf[(size_t)ch * nx + o];
}

// S2 projection of the z2 block of nonleaf i after the step z - alpha L* eta,
// and s^0 - alpha at the root. Closed form of the projection on the kernel of
// G = [aI, -I, 1, -I, -I]: (G G')^{-1} = (I - 11'/(c+n))/c, c = a^2 + 3.
template <typename S, int T, int D = kMaxDim>
__device__ __forceinline__ void fam_s2(const DevProb<S>& P, const Off<S>& O, const S* __restrict__ z,
                                       const S* __restrict__ eta, S* __restrict__ zout, int i,
                                       int lane) {
  const int nx = P.nx, nu = P.nu, fc = P.fc[i], n = P.nch[i];
  const S al = P.alpha;
  const long long zb = O.z2(i);
  const long long e1 = O.e1(i);
  const S es = eta[O.e1s(i)];
  const S a = P.a[i];
  const S y3h = z[zb + 2 * n] - al * (eta[e1 + 2 * n] - es);
  double gsum = 0;
  for (int pass = 0; pass < 2; ++pass) {
    const S cc = a * a + S(3);
    const S Gs = pass ? (S)team_sum<T>(gsum) : S(0);
    double wsum = 0;
    for (int k = lane; k < n; k += T) {
      const int ch = fc + k;
      const S y1h = z[zb + k] - al * (eta[e1 + k] - P.p[ch] * es);
      const S y2h = z[zb + n + k] - al * eta[e1 + n + k];
      const long long e2c = O.e2(ch) + nx + nu;
      const S th = z[zb + 2 * n + 1 + k] - al * S(0.5) * (eta[e2c] + eta[e2c + 1]);
      S Lts;
      if (ch < P.nl) {
        Lts = eta[O.e1s(ch)];
      } else {
        const long long e3c = O.e3(ch) + 2 * nx;
        Lts = S(0.5) * (eta[e3c] + eta[e3c + 1]);
      }
      const S sh = z[zb + 3 * n + 1 + k] - al * Lts;
      const S g = a * y1h - y2h + y3h - th - sh;
      if (!pass) {
        gsum += (double)g;
      } else {
        const S w = (g - Gs / (cc + S(n))) / cc;
        wsum += (double)w;
        zout[zb + k] = y1h - a * w;
        zout[zb + n + k] = y2h + w;
        zout[zb + 2 * n + 1 + k] = th + w;
        zout[zb + 3 * n + 1 + k] = sh + w;
      }
    }
    if (pass) {
      const S Ws = (S)team_sum<T>(wsum);
      if (lane == 0) {
        zout[zb + 2 * n] = y3h - Ws;
        if (i == 0) zout[0] = z[0] - al * es - al;
      }
    }
  }
}

// Dual update and residual statistics of the rows of child ch (group 2, and
// group 3 if ch is a leaf) and of the columns tau^ch (and x^ch, s^ch at a
// leaf). xp/xo: x+^i and x^i (lane chunks); vu: u+^i in LDS; xc: x+^ch (lane
// chunks); vr: LDS scratch of 2*VM; gx, gu accumulate the group-2 part of
// L* r_eta on columns x^i, u^i.
template <typename S, int T, int D = kMaxDim>
__device__ __forceinline__ void fam_dual_child(const DevProb<S>& P, const Off<S>& O,
                                               const S* __restrict__ z, const S* __restrict__ eta,
                                               const S* __restrict__ zout, S* __restrict__ eout, int i,
                                               int ch, int lane, const S (&xp)[(D + T - 1) / T],
                                               const S (&xo)[(D + T - 1) / T], const S* vu,
                                               const S (&xc)[(D + T - 1) / T], S* vr,
                                               S (&gx)[(D + T - 1) / T],
                                               S (&gu)[(D + T - 1) / T], StatAcc& st) {
  constexpr int C = (D + T - 1) / T;
  constexpr int C2 = (2 * D + T - 1) / T;
  const int nx = P.nx, nu = P.nu;
  const S al = P.alpha;
  const S ia = S(1) / al;
  const long long ui = O.u(i);
  // ---- group 2: (Q^{1/2} x^i, R^{1/2} u^i, tau/2, tau/2) in SOC + shift
  const long long e2 = O.e2(ch);
  const long long tpos = O.tau(ch);
  const S tau = z[tpos], taup = zout[tpos];
  S wv[C2], ov[C2], lz[C2];
#pragma unroll
  for (int c = 0; c < C2; ++c) {
    const int o = lane + c * T;
    wv[c] = 0;
    ov[c] = 0;
    lz[c] = 0;
    if (o < nx) {
      const S xpo = xp[c < C ? c : C - 1], xoo = xo[c < C ? c : C - 1];
      const S sqv = P.sq[(size_t)ch * nx + o];
      wv[c] = eta[e2 + o] + al * sqv * (S(2) * xpo - xoo);
      lz[c] = sqv * (xoo - xpo);
    } else if (o < nx + nu) {
      const int ou = o - nx;
      const S upo = vu[ou], uoo = z[ui + ou];
      const S srv = P.sr[(size_t)ch * nu + ou];
      wv[c] = eta[e2 + o] + al * srv * (S(2) * upo - uoo);
      lz[c] = srv * (uoo - upo);
    }
  }
  const S wa = eta[e2 + nx + nu] + al * S(0.5) * (S(2) * taup - tau);
  const S wb = eta[e2 + nx + nu + 1] + al * S(0.5) * (S(2) * taup - tau);
  S oa, ob;
  soc_prox<S, T, D>(wv, ov, nx + nu, wa, wb, oa, ob, al, lane);
  const S rtau = tau - taup;
#pragma unroll
  for (int c = 0; c < C2; ++c) {
    const int o = lane + c * T;
    if (o < nx + nu) {
      eout[e2 + o] = ov[c];
      const S re = eta[e2 + o] - ov[c];
      vr[o] = re;
      st.row((double)re, (double)lz[c], (double)ia);
    }
  }
  wave_lds_sync();
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    if (o < nx) gx[c] += P.sq[(size_t)ch * nx + o] * vr[o];
    if (o < nu) gu[c] += P.sr[(size_t)ch * nu + o] * vr[nx + o];
  }
  wave_lds_sync();
  if (lane == 0) {
    const S rea = eta[e2 + nx + nu] - oa, reb = eta[e2 + nx + nu + 1] - ob;
    eout[e2 + nx + nu] = oa;
    eout[e2 + nx + nu + 1] = ob;
    st.row((double)rea, 0.5 * (double)rtau, (double)ia);
    st.row((double)reb, 0.5 * (double)rtau, (double)ia);
    st.col((double)rtau, 0.5 * ((double)rea + (double)reb), (double)ia);
  }
  if (ch < P.nl) return;
  // ---- group 3 of a leaf: box on x, (Q_N^{1/2} x, s/2, s/2) in SOC + shift
  const long long e3 = O.e3(ch);
  const long long spos = O.s(ch);
  const S sv = z[spos], svp = zout[spos];
  S wq[C2], oq[C2];
  S rex[C], xin[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    rex[c] = 0;
    xin[c] = 0;
    if (o < nx) {
      const S xcin = z[O.x(ch) + o];
      xin[c] = xcin;
      const S wbx = eta[e3 + o] + al * (S(2) * xc[c] - xcin);
      const S pb = wbx - al * clampv(wbx * ia, P.xlo[(size_t)ch * nx + o], P.xhi[(size_t)ch * nx + o]);
      eout[e3 + o] = pb;
      rex[c] = eta[e3 + o] - pb;
      st.row((double)rex[c], (double)(xcin - xc[c]), (double)ia);
    }
  }
#pragma unroll
  for (int c = 0; c < C2; ++c) {
    const int o = lane + c * T;
    wq[c] = 0;
    oq[c] = 0;
    if (c < C && o < nx) {
      const int cc = c < C ? c : C - 1;
      wq[c] = eta[e3 + nx + o] + al * P.sqN[(size_t)ch * nx + o] * (S(2) * xc[cc] - xin[cc]);
    }
  }
  const S wsa = eta[e3 + 2 * nx] + al * S(0.5) * (S(2) * svp - sv);
  const S wsb = eta[e3 + 2 * nx + 1] + al * S(0.5) * (S(2) * svp - sv);
  S osa, osb;
  soc_prox<S, T, D>(wq, oq, nx, wsa, wsb, osa, osb, al, lane);
  const S rs = sv - svp;
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    if (o < nx) {
      eout[e3 + nx + o] = oq[c];
      const S reqv = eta[e3 + nx + o] - oq[c];
      const S sqn = P.sqN[(size_t)ch * nx + o];
      st.row((double)reqv, (double)(sqn * (xin[c] - xc[c])), (double)ia);
      // column x^ch of a leaf: L* r_eta = r_eta(box) + Q_N^{1/2} r_eta(q)
      st.col((double)(xin[c] - xc[c]), (double)(rex[c] + sqn * reqv), (double)ia);
    }
  }
  if (lane == 0) {
    eout[e3 + 2 * nx] = osa;
    eout[e3 + 2 * nx + 1] = osb;
    const S rea3 = eta[e3 + 2 * nx] - osa, reb3 = eta[e3 + 2 * nx + 1] - osb;
    st.row((double)rea3, 0.5 * (double)rs, (double)ia);
    st.row((double)reb3, 0.5 * (double)rs, (double)ia);
    st.col((double)rs, 0.5 * ((double)rea3 + (double)reb3), (double)ia);
  }
}

// Dual update of group 1 of nonleaf i: y in K* = R^{2n}_+ x R, s - b'y in
// R_+, (x, u) in the box; columns y^i, s^i, x^i, u^i of L* r_eta.
template <typename S, int T, int D = kMaxDim>
__device__ __forceinline__ void fam_dual_node(const DevProb<S>& P, const Off<S>& O,
                                              const S* __restrict__ z, const S* __restrict__ eta,
                                              const S* __restrict__ zout, S* __restrict__ eout, int i,
                                              int lane, const S (&xp)[(D + T - 1) / T],
                                              const S (&xo)[(D + T - 1) / T],
                                              const S (&up)[(D + T - 1) / T],
                                              const S (&uo)[(D + T - 1) / T],
                                              const S (&gx)[(D + T - 1) / T],
                                              const S (&gu)[(D + T - 1) / T], StatAcc& st) {
  constexpr int C = (D + T - 1) / T;
  const int nx = P.nx, nu = P.nu, fc = P.fc[i], n = P.nch[i];
  const S al = P.alpha;
  const S ia = S(1) / al;
  const long long zb = O.z2(i);
  const long long e1 = O.e1(i);
  const long long spos = O.s(i);
  const S si = z[spos], sip = zout[spos];
  double bw = 0, bry = 0;
  for (int k = lane; k < n; k += T) {
    const S pk = P.p[fc + k];
    const S y1 = z[zb + k], y1p = zout[zb + k];
    bw += (double)(pk * (S(2) * y1p - y1));
    bry += (double)(pk * (y1 - y1p));
  }
  const S y3 = z[zb + 2 * n], y3p = zout[zb + 2 * n];
  const S bW = (S)team_sum<T>(bw) + (S(2) * y3p - y3);
  const S bR = (S)team_sum<T>(bry) + (y3 - y3p);
  const S ws = eta[e1 + 2 * n + 1] + al * ((S(2) * sip - si) - bW);
  const S es_new = ws < S(0) ? ws : S(0);
  const S res_ = eta[e1 + 2 * n + 1] - es_new;
  for (int k = lane; k < 2 * n + 1; k += T) {
    const S y = z[zb + k], yp = zout[zb + k];
    const S w = eta[e1 + k] + al * (S(2) * yp - y);
    const S ep = (k < 2 * n) ? (w < S(0) ? w : S(0)) : S(0);
    eout[e1 + k] = ep;
    const S re = eta[e1 + k] - ep;
    const S ry = y - yp;
    st.row((double)re, (double)ry, (double)ia);
    const S bk = (k < n) ? P.p[fc + k] : ((k == 2 * n) ? S(1) : S(0));
    st.col((double)ry, (double)(re - bk * res_), (double)ia);
  }
  if (lane == 0) {
    eout[e1 + 2 * n + 1] = es_new;
    const S rsi = si - sip;
    st.row((double)res_, (double)(rsi - bR), (double)ia);
    st.col((double)rsi, (double)res_, (double)ia);
  }
  const long long e1x = O.e1x(i), e1u = O.e1u(i);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    if (o < nx) {
      const S w = eta[e1x + o] + al * (S(2) * xp[c] - xo[c]);
      const S ep = w - al * clampv(w * ia, P.xlo[(size_t)i * nx + o], P.xhi[(size_t)i * nx + o]);
      eout[e1x + o] = ep;
      const S re = eta[e1x + o] - ep;
      const S rz = xo[c] - xp[c];
      st.row((double)re, (double)rz, (double)ia);
      st.col((double)rz, (double)(re + gx[c]), (double)ia);
    }
    if (o < nu) {
      const S w = eta[e1u + o] + al * (S(2) * up[c] - uo[c]);
      const S ep = w - al * clampv(w * ia, P.ulo[(size_t)i * nu + o], P.uhi[(size_t)i * nu + o]);
      eout[e1u + o] = ep;
      const S re = eta[e1u + o] - ep;
      const S rz = uo[c] - up[c];
      st.row((double)re, (double)rz, (double)ia);
      st.col((double)rz, (double)(re + gu[c]), (double)ia);
    }
  }
}

// Fixed-order block reduction of the statistics into one partial record.
__device__ __forceinline__ void block_stats(const StatAcc& st, double* __restrict__ partials) {
  __shared__ double red[kStats][256];
  red[0][threadIdx.x] = st.rz2;
  red[1][threadIdx.x] = st.re2;
  red[2][threadIdx.x] = st.cross;
  red[3][threadIdx.x] = st.xip;
  red[4][threadIdx.x] = st.xid;
  __syncthreads();
  for (int s = blockDim.x / 2; s >= 1; s >>= 1) {
    if ((int)threadIdx.x < s) {
      red[0][threadIdx.x] += red[0][threadIdx.x + s];
      red[1][threadIdx.x] += red[1][threadIdx.x + s];
      red[2][threadIdx.x] += red[2][threadIdx.x + s];
      red[3][threadIdx.x] = fmax(red[3][threadIdx.x], red[3][threadIdx.x + s]);
      red[4][threadIdx.x] = fmax(red[4][threadIdx.x], red[4][threadIdx.x + s]);
    }
    __syncthreads();
  }
  if (threadIdx.x < kStats) partials[(size_t)blockIdx.x * kStats + threadIdx.x] = red[threadIdx.x][0];
}

// Backward step of nonleaf i by one team (Alg. 2 backward sweep with
// W = sum_c Abar^c' P^c B^c): d = R~^{-1}(ubar - sum_c B^c' q^c),
// q = K'(d - ubar) + W d - xbar + sum_c Abar^c' q^c. LDS: 3 VM per team.
template <typename S, int T, int D = kMaxDim>
__device__ __forceinline__ void fam_bwd_team(const DevProb<S>& P, const S* __restrict__ xbar,
                                             const S* __restrict__ ubar, S* __restrict__ qbuf,
                                             S* __restrict__ dbuf, int i, int lane, S* lds, int VM) {
  constexpr int C = (D + T - 1) / T;
  S* vq = lds;
  S* vg = vq + VM;
  S* vd = vg + VM;
  const int nx = P.nx, nu = P.nu;
  const int fc = P.fc[i], n = P.nch[i];
  S xb[C], ub[C], sA[C], h[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    xb[c] = (o < nx) ? xbar[(size_t)i * nx + o] : S(0);
    ub[c] = (o < nu) ? ubar[(size_t)i * nu + o] : S(0);
    sA[c] = h[c] = 0;
  }
  for (int k = 0; k < n; ++k) {
    const int ch = fc + k;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int o = lane + c * T;
      if (o < nx) vq[o] = qbuf[(size_t)ch * nx + o];
    }
    wave_lds_sync();
    mv_acc<S, T, D>(h, P.BR + (size_t)ch * nx * nu, nx, nu, vq, lane);
    mv_acc<S, T, D>(sA, P.AbR + (size_t)ch * nx * nx, nx, nx, vq, lane);
    wave_lds_sync();
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    if (o < nu) vg[o] = ub[c] - h[c];
  }
  wave_lds_sync();
  S dv[C];
#pragma unroll
  for (int c = 0; c < C; ++c) dv[c] = 0;
  mv_acc<S, T, D>(dv, P.Rinv + (size_t)i * nu * nu, nu, nu, vg, lane);
  wave_lds_sync();
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    if (o < nu) {
      vg[o] = dv[c] - ub[c];
      vd[o] = dv[c];
      dbuf[(size_t)i * nu + o] = dv[c];
    }
  }
  wave_lds_sync();
  S qi[C];
#pragma unroll
  for (int c = 0; c < C; ++c) qi[c] = sA[c] - xb[c];
  mv_acc<S, T, D>(qi, P.KR + (size_t)i * nu * nx, nu, nx, vg, lane);
  mv_acc<S, T, D>(qi, P.WC + (size_t)i * nu * nx, nu, nx, vd, lane);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    if (o < nx) qbuf[(size_t)i * nx + o] = qi[c];
  }
  wave_lds_sync();
}

// Forward step of nonleaf i by one team (Alg. 2 forward sweep):
// u = K x + d, x^c = Abar^c x + B^c d; x^0 = x0 at the root. LDS: 2 VM.
template <typename S, int T, int D = kMaxDim>
__device__ __forceinline__ void fam_fwd_team(const DevProb<S>& P, S* __restrict__ zout,
                                             const S* __restrict__ dbuf, const double* __restrict__ x0,
                                             int i, int lane, S* lds, int VM) {
  constexpr int C = (D + T - 1) / T;
  S* vx = lds;
  S* vd = vx + VM;
  const Off<S> O(P);
  const int nx = P.nx, nu = P.nu;
  const int fc = P.fc[i], n = P.nch[i];
  const long long ui = O.u(i);
  S up[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    up[c] = 0;
    if (o < nx) {
      S xv;
      if (i == 0) {
        xv = (S)x0[o];
        zout[1 + o] = xv;
      } else {
        xv = zout[O.x(i) + o];
      }
      vx[o] = xv;
    }
    if (o < nu) {
      const S dd = dbuf[(size_t)i * nu + o];
      vd[o] = dd;
      up[c] = dd;
    }
  }
  wave_lds_sync();
  mv_acc<S, T, D>(up, P.KC + (size_t)i * nx * nu, nx, nu, vx, lane);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    if (o < nu) zout[ui + o] = up[c];
  }
  for (int k = 0; k < n; ++k) {
    const int ch = fc + k;
    S xc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) xc[c] = 0;
    mv_acc<S, T, D>(xc, P.AbC + (size_t)ch * nx * nx, nx, nx, vx, lane);
    mv_acc<S, T, D>(xc, P.BC + (size_t)ch * nu * nx, nu, nx, vd, lane);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int o = lane + c * T;
      if (o < nx) zout[O.x(ch) + o] = xc[c];
    }
  }
  wave_lds_sync();
}

// pre-pass of family i by one team: xbar, ubar; leaf children's q = -xbar;
// S2 projection of the z2 block; s^0 - alpha at the root.
template <typename S, int T, int D = kMaxDim>
__device__ __forceinline__ void fam_pre_team(const DevProb<S>& P, const S* __restrict__ z,
                                             const S* __restrict__ eta, S* __restrict__ zout,
                                             S* __restrict__ xbar, S* __restrict__ ubar,
                                             S* __restrict__ qbuf, int i, int lane) {
  constexpr int C = (D + T - 1) / T;
  const Off<S> O(P);
  const int nx = P.nx, nu = P.nu, fc = P.fc[i], n = P.nch[i];
  S xb[C], ub[C];
  fam_xbar_ubar<S, T, D>(P, O, z, eta, i, lane, xb, ub);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    if (o < nx) xbar[(size_t)i * nx + o] = xb[c];
    if (o < nu) ubar[(size_t)i * nu + o] = ub[c];
  }
  if (fc >= P.nl) {  // children are leaves
    for (int k = 0; k < n; ++k)
      for (int o = lane; o < nx; o += T)
        qbuf[(size_t)(fc + k) * nx + o] = fam_child_q<S>(P, O, z, eta, qbuf, fc + k, o);
  }
  fam_s2<S, T, D>(P, O, z, eta, zout, i, lane);
}

// post-pass of family i by one team: dual update and residual statistics.
// LDS: 3 VM per team.
template <typename S, int T, int D = kMaxDim>
__device__ __forceinline__ void fam_post_team(const DevProb<S>& P, const S* __restrict__ z,
                                              const S* __restrict__ eta, const S* __restrict__ zout,
                                              S* __restrict__ eout, int i, int lane, S* lds, int VM,
                                              StatAcc& st) {
  constexpr int C = (D + T - 1) / T;
  S* vu = lds;
  S* vr = vu + VM;
  const Off<S> O(P);
  const int nx = P.nx, nu = P.nu, fc = P.fc[i], n = P.nch[i];
  const long long ui = O.u(i);
  S xp[C], xo[C], up[C], uo[C], gx[C], gu[C];
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const int o = lane + c * T;
    xp[c] = xo[c] = up[c] = uo[c] = gx[c] = gu[c] = 0;
    if (o < nx) {
      xp[c] = zout[O.x(i) + o];
      xo[c] = z[O.x(i) + o];
    }
    if (o < nu) {
      up[c] = zout[ui + o];
      uo[c] = z[ui + o];
      vu[o] = up[c];
    }
  }
  wave_lds_sync();
  for (int k = 0; k < n; ++k) {
    const int ch = fc + k;
    S xc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const int o = lane + c * T;
      xc[c] = (o < nx) ? zout[O.x(ch) + o] : S(0);
    }
    fam_dual_child<S, T, D>(P, O, z, eta, zout, eout, i, ch, lane, xp, xo, vu, xc, vr, gx, gu, st);
  }
  fam_dual_node<S, T, D>(P, O, z, eta, zout, eout, i, lane, xp, xo, up, uo, gx, gu, st);
  wave_lds_sync();
}

// Pre-pass of a family by a team: b[s] = component lane + T s of (xbar, ubar)
// = (x, u) - alpha L* eta; the (y, tau, s) block's step and its projection on
// S2 (closed form, as fam_s2), held in registers between its two sums while
// n <= T; s^0 - alpha at the root.
template <typename S, int T, int SL, typename IX>
__device__ __forceinline__ void flat_pre_family(const DevProb<S>& P, const Off<S, IX>& O, const S* __restrict__ z,
                                                const S* __restrict__ eta, S* __restrict__ zout, int i, int fc, int n,
                                                int lane, S (&b)[SL]) {
  const int nx = P.nx, nu = P.nu, K = nx + nu;
  const S al = P.alpha;
  const IX e1 = (IX)2 * (fc - 1) + (IX)i * (2 + K), e1s = e1 + 2 * n + 1;
  const IX zb = (IX)P.zZ2 + (IX)4 * (fc - 1) + i, e2 = O.e2(fc);
  // One batch of loads, without branches around them (clamped indices): the
  // y block's operands (child `lane`) and the columns x^i, u^i with the first
  // child; the next child's are in flight while one is added.
  const S es = at<S, IX>(eta, e1s), a = at<S, IX>(P.a, i), y3 = at<S, IX>(z, zb + 2 * n), ey3 = at<S, IX>(eta, e1 + 2 * n);
  const bool leaf = fc >= P.nl;
  struct Slack {
    S z1, z2, zt, zs, e1, e2, p, ta, tb, sa, sb;
  };
  auto load = [&](int k, Slack& w) {
    const IX e = e2 + (IX)k * (K + 2) + K;
    const IX sa = leaf ? O.e3(fc + k) + 2 * nx : O.e1s(leaf ? 0 : fc + k);
    w.sa = at<S, IX>(eta, sa);
    w.sb = at<S, IX>(eta, leaf ? sa + 1 : sa);
    w.ta = at<S, IX>(eta, e);
    w.tb = at<S, IX>(eta, e + 1);
    w.z1 = at<S, IX>(z, zb + k);
    w.z2 = at<S, IX>(z, zb + n + k);
    w.zt = at<S, IX>(z, zb + 2 * n + 1 + k);
    w.zs = at<S, IX>(z, zb + 3 * n + 1 + k);
    w.e1 = at<S, IX>(eta, e1 + k);
    w.e2 = at<S, IX>(eta, e1 + n + k);
    w.p = at<S, IX>(P.p, fc + k);
  };
  auto step = [&](const Slack& w, S& y1h, S& y2h, S& th, S& sh) {
    y1h = w.z1 - al * (w.e1 - w.p * es);
    y2h = w.z2 - al * w.e2;
    th = w.zt - al * S(0.5) * (w.ta + w.tb);
    sh = w.zs - al * (leaf ? S(0.5) * (w.sa + w.sb) : w.sa);
  };
  Slack mine;
  load(lane < n ? lane : n - 1, mine);
  S zv[SL], acc[SL], cs[SL], ce[SL];
  const S* sc[SL];
  IX so[SL];
  int kk[SL];
#pragma unroll
  for (int s = 0; s < SL; ++s) {
    const int k = lane + T * s;
    kk[s] = k < K ? k : 0;
    const bool isx = kk[s] < nx;
    so[s] = (IX)fc * (isx ? nx : nu) + (isx ? kk[s] : kk[s] - nx);
    sc[s] = pair_base<S, IX>(P.sq, P.sr, isx, so[s]);
    zv[s] = at<S, IX>(z, isx ? O.x(i) + kk[s] : O.u(i) + (kk[s] - nx));
    acc[s] = at<S, IX>(eta, e1s + 1 + kk[s]);
    cs[s] = at<S, IX>(sc[s], so[s]);
    ce[s] = at<S, IX>(eta, e2 + kk[s]);
  }
  for (int c = 0; c < n; ++c) {
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      const S f = cs[s], g = ce[s];
      if (c + 1 < n) {
        so[s] += kk[s] < nx ? nx : nu;
        cs[s] = at<S, IX>(sc[s], so[s]);
        ce[s] = at<S, IX>(eta, e2 + (IX)(c + 1) * (K + 2) + kk[s]);
      }
      acc[s] += f * g;
    }
  }
#pragma unroll
  for (int s = 0; s < SL; ++s) b[s] = zv[s] - al * acc[s];
  S y1h, y2h, th, sh;
  step(mine, y1h, y2h, th, sh);
  // ---- S2
  const S y3h = y3 - al * (ey3 - es);
  const S cc = a * a + S(3);
  auto g_of = [&](S y1, S y2, S t, S s) { return a * y1 - y2 + y3h - t - s; };
  double gsum = lane < n ? (double)g_of(y1h, y2h, th, sh) : 0.0;
  for (int k = lane + T; k < n; k += T) {
    S p, q, t, s;
    Slack w;
    load(k, w);
    step(w, p, q, t, s);
    gsum += (double)g_of(p, q, t, s);
  }
  const S corr = (S)team_sum<T>(gsum) / (cc + S(n));
  double wsum = 0;
  auto store = [&](int k, S y1, S y2, S t, S s) {
    const S w = (g_of(y1, y2, t, s) - corr) / cc;
    wsum += (double)w;
    at<S, IX>(zout, zb + k) = y1 - a * w;
    at<S, IX>(zout, zb + n + k) = y2 + w;
    at<S, IX>(zout, zb + 2 * n + 1 + k) = t + w;
    at<S, IX>(zout, zb + 3 * n + 1 + k) = s + w;
  };
  for (int k = lane + T; k < n; k += T) {  // more than T children
    S p, q, t, s;
    Slack w;
    load(k, w);
    step(w, p, q, t, s);
    store(k, p, q, t, s);
  }
  if (lane < n) store(lane, y1h, y2h, th, sh);
  const S Ws = (S)team_sum<T>(wsum);
  if (lane == 0) {
    at<S, IX>(zout, zb + 2 * n) = y3h - Ws;
    if (i == 0) at<S, IX>(zout, 0) = at<S, IX>(z, 0) - al * es - al;
  }
}

// Flat forms of the passes: a team of T lanes (T <= 64, inside one wavefront)
// owns a unit, a nonleaf family (group 1 of i and group 2 of each child c) or
// a leaf (group 3). The rows and columns a unit touches are exactly those of
// the family-serial form, so no unit waits on another. A family's columns
// x^i and u^i share one index k < nx + nu <= T SL with the first rows of each
// child's group 2, so every lane holds the same SL components of all of them.
// Offsets are arithmetic in i once fc = fc[i], n = nch[i] and the slot sp of
// s^i in its ancestor's block are known: one level of index loads, then every
// data load of the unit at once. zp_at(kk): component kk of (x+, u+).
template <typename S, int T, int SL, typename IX, typename F>
__device__ __forceinline__ void flat_family(const DevProb<S>& P, const Off<S, IX>& O, IX sp,
                                            const S* __restrict__ z, const S* __restrict__ eta,
                                            const S* __restrict__ zout, S* __restrict__ eout, int i, int fc, int n,
                                            int lane, F&& zp_at, StatAcc& st) {
  const int nx = P.nx, nu = P.nu, K = nx + nu;
  const S al = P.alpha;
  const S ia = S(1) / al;
  const IX e1 = (IX)2 * (fc - 1) + (IX)i * (2 + K), e1x = e1 + 2 * n + 2, zb = (IX)P.zZ2 + (IX)4 * (fc - 1) + i;
  const IX xi = O.x(i), ui = O.u(i);
  // One batch of loads, with clamped indices and no branches, so that
  // every load of the unit is in flight at once: columns x^i, u^i (slot s:
  // k = lane + 64 s), the y block (one entry per lane when 2n + 1 <= T)
  // and the scalars.
  // FP64 loads the box rows' and the y block's operands after the cone
  // blocks at two components a lane (fewer live registers across them)
  constexpr bool kLateBox = sizeof(S) == 8 && SL > 1;
  bool on[SL];
  S zp[SL], zo[SL], lo[SL], hi[SL], eb[SL], gc[SL];
  auto load_box = [&](int s) {
    const int k = lane + T * s;
    const int kk = on[s] ? k : 0;
    const bool isx = kk < nx;
    const IX bi = isx ? (IX)i * nx + kk : (IX)i * nu + (kk - nx);
    IX bl = bi, bh = bi;
    const S* plo = pair_base<S, IX>(P.xlo, P.ulo, isx, bl);
    const S* phi = pair_base<S, IX>(P.xhi, P.uhi, isx, bh);
    lo[s] = at<S, IX>(plo, bl);
    hi[s] = at<S, IX>(phi, bh);
    eb[s] = at<S, IX>(eta, e1x + kk);
  };
#pragma unroll
  for (int s = 0; s < SL; ++s) {
    const int k = lane + T * s;
    on[s] = k < K;
    const int kk = on[s] ? k : 0;
    const bool isx = kk < nx;
    const IX zi = isx ? xi + kk : ui + (kk - nx);
    zp[s] = zp_at(kk);
    zo[s] = at<S, IX>(z, zi);
    if (!kLateBox) load_box(s);
    gc[s] = 0;
  }
  const int ny = 2 * n + 1;
  const int ky = lane < ny ? lane : 0;
  S yv, ypv, eyv, pk, si, sip, y3, y3p, es;
  auto load_y = [&]() {
    yv = at<S, IX>(z, zb + ky);
    ypv = at<S, IX>(zout, zb + ky);
    eyv = at<S, IX>(eta, e1 + ky);
    pk = at<S, IX>(P.p, fc + (lane < n ? lane : 0));
    si = at<S, IX>(z, sp);
    sip = at<S, IX>(zout, sp);
    y3 = at<S, IX>(z, zb + 2 * n);
    y3p = at<S, IX>(zout, zb + 2 * n);
    es = at<S, IX>(eta, e1 + 2 * n + 1);
  };
  if (!kLateBox) load_y();
  // group 2 of every child: (Q^{1/2} x^i, R^{1/2} u^i, tau/2, tau/2); at one
  // component a lane the next child's operands are in flight meanwhile
  struct Child {
    S sc[SL], ev[SL], tau, taup, ea, ebb;
  };
  auto load_child = [&](int c, Child& C) {
    const IX e2 = O.e2(c);
    const IX tp = zb + 2 * n + 1 + (c - fc);
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      const int kk = on[s] ? lane + T * s : 0;
      IX so = kk < nx ? (IX)c * nx + kk : (IX)c * nu + (kk - nx);
      const S* ps = pair_base<S, IX>(P.sq, P.sr, kk < nx, so);
      C.sc[s] = at<S, IX>(ps, so);
      C.ev[s] = at<S, IX>(eta, e2 + kk);
    }
    C.tau = at<S, IX>(z, tp);
    C.taup = at<S, IX>(zout, tp);
    C.ea = at<S, IX>(eta, e2 + K);
    C.ebb = at<S, IX>(eta, e2 + K + 1);
  };
  Child nxt;
  if (SL == 1) load_child(fc, nxt);
  for (int c = fc; c < fc + n; ++c) {
    const IX e2 = O.e2(c);
    if (SL > 1) load_child(c, nxt);
    const Child C = nxt;
    if (SL == 1 && c + 1 < fc + n) load_child(c + 1, nxt);
    const S(&sc)[SL] = C.sc;
    const S(&ev)[SL] = C.ev;
    const S tau = C.tau, taup = C.taup, ea = C.ea, ebb = C.ebb;
    S wv[SL], ov[SL], lz[SL];
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      wv[s] = on[s] ? ev[s] + al * sc[s] * (S(2) * zp[s] - zo[s]) : S(0);
      lz[s] = sc[s] * (zo[s] - zp[s]);
      ov[s] = 0;
    }
    const S wa = ea + al * S(0.5) * (S(2) * taup - tau);
    const S wb = ebb + al * S(0.5) * (S(2) * taup - tau);
    S oa, ob;
    soc_prox<S, T, T * SL / 2>(wv, ov, K, wa, wb, oa, ob, al, lane);
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      if (on[s]) {
        at<S, IX>(eout, e2 + lane + T * s) = ov[s];
        const S re = ev[s] - ov[s];
        st.row((double)re, (double)lz[s], (double)ia);
        gc[s] += sc[s] * re;
      }
    }
    if (lane == 0) {
      const S rtau = tau - taup;
      const S rea = ea - oa, reb = ebb - ob;
      at<S, IX>(eout, e2 + K) = oa;
      at<S, IX>(eout, e2 + K + 1) = ob;
      st.row((double)rea, 0.5 * (double)rtau, (double)ia);
      st.row((double)reb, 0.5 * (double)rtau, (double)ia);
      st.col((double)rtau, 0.5 * ((double)rea + (double)reb), (double)ia);
    }
  }
  // group 1: the boxes on (x^i, u^i) and the columns x^i, u^i
  if (kLateBox) {
#pragma unroll
    for (int s = 0; s < SL; ++s) load_box(s);
    load_y();
  }
#pragma unroll
  for (int s = 0; s < SL; ++s) {
    if (on[s]) {
      const S w = eb[s] + al * (S(2) * zp[s] - zo[s]);
      const S ep = w - al * clampv(w * ia, lo[s], hi[s]);
      at<S, IX>(eout, e1x + lane + T * s) = ep;
      const S re = eb[s] - ep;
      const S rz = zo[s] - zp[s];
      st.row((double)re, (double)rz, (double)ia);
      st.col((double)rz, (double)(re + gc[s]), (double)ia);
    }
  }
  // group 1: y in K* = R^{2n}_+ x R and the row s^i - b'y
  double bw = lane < n ? (double)(pk * (S(2) * ypv - yv)) : 0.0;
  double bry = lane < n ? (double)(pk * (yv - ypv)) : 0.0;
  for (int k = lane + T; k < n; k += T) {  // more than T children
    const S pq = at<S, IX>(P.p, fc + k);
    const S y1 = at<S, IX>(z, zb + k), y1p = at<S, IX>(zout, zb + k);
    bw += (double)(pq * (S(2) * y1p - y1));
    bry += (double)(pq * (y1 - y1p));
  }
  const S bW = (S)team_sum<T>(bw) + (S(2) * y3p - y3);
  const S bR = (S)team_sum<T>(bry) + (y3 - y3p);
  const S ws = es + al * ((S(2) * sip - si) - bW);
  const S es_new = ws < S(0) ? ws : S(0);
  const S res_ = es - es_new;
  auto yrow = [&](int k, S y, S yp, S e, S pq) {
    const S w = e + al * (S(2) * yp - y);
    const S ep = (k < 2 * n) ? (w < S(0) ? w : S(0)) : S(0);
    at<S, IX>(eout, e1 + k) = ep;
    const S re = e - ep;
    const S ry = y - yp;
    st.row((double)re, (double)ry, (double)ia);
    const S bk = (k < n) ? pq : ((k == 2 * n) ? S(1) : S(0));
    st.col((double)ry, (double)(re - bk * res_), (double)ia);
  };
  if (lane < ny) yrow(lane, yv, ypv, eyv, pk);
  for (int k = lane + T; k < ny; k += T) yrow(k, at<S, IX>(z, zb + k), at<S, IX>(zout, zb + k), at<S, IX>(eta, e1 + k), k < n ? at<S, IX>(P.p, fc + k) : S(0));
  if (lane == 0) {
    at<S, IX>(eout, e1 + 2 * n + 1) = es_new;
    const S rsi = si - sip;
    st.row((double)res_, (double)(rsi - bR), (double)ia);
    st.col((double)rsi, (double)res_, (double)ia);
  }
}

// Leaf j: group 3 (box on x^j, (Q_N^{1/2} x^j, s/2, s/2) in the SOC) and
// the columns x^j, s^j; one batch of loads as in flat_family.
// n_x <= T SL; xp_at(o): component o of x+^j.
template <typename S, int T, int SL, typename IX, typename F>
__device__ __forceinline__ void flat_leaf(const DevProb<S>& P, const Off<S, IX>& O, IX sp,
                                          const S* __restrict__ z, const S* __restrict__ eta,
                                          const S* __restrict__ zout, S* __restrict__ eout, int j, int lane,
                                          F&& xp_at, StatAcc& st) {
  const int nx = P.nx;
  const S al = P.alpha;
  const S ia = S(1) / al;
  const IX e3 = O.e3(j), xj = O.x(j);
  S xc[SL], xin[SL], ebx[SL], eq[SL], lo[SL], hi[SL], sqn[SL];
  bool on[SL];
#pragma unroll
  for (int s = 0; s < SL; ++s) {
    on[s] = lane + T * s < nx;
    const int kk = on[s] ? lane + T * s : 0;
    xc[s] = xp_at(kk);
    xin[s] = at<S, IX>(z, xj + kk);
    ebx[s] = at<S, IX>(eta, e3 + kk);
    eq[s] = at<S, IX>(eta, e3 + nx + kk);
    lo[s] = at<S, IX>(P.xlo, (IX)j * nx + kk);
    hi[s] = at<S, IX>(P.xhi, (IX)j * nx + kk);
    sqn[s] = at<S, IX>(P.sqN, (IX)j * nx + kk);
  }
  const S sv = at<S, IX>(z, sp), svp = at<S, IX>(zout, sp);
  const S ea = at<S, IX>(eta, e3 + 2 * nx), ebb = at<S, IX>(eta, e3 + 2 * nx + 1);
  S wq[SL], oq[SL];
#pragma unroll
  for (int s = 0; s < SL; ++s) {
    wq[s] = on[s] ? eq[s] + al * sqn[s] * (S(2) * xc[s] - xin[s]) : S(0);
    oq[s] = 0;
  }
  const S wsa = ea + al * S(0.5) * (S(2) * svp - sv);
  const S wsb = ebb + al * S(0.5) * (S(2) * svp - sv);
  S osa, osb;
  soc_prox<S, T, T * SL / 2>(wq, oq, nx, wsa, wsb, osa, osb, al, lane);
#pragma unroll
  for (int s = 0; s < SL; ++s) {
    if (!on[s]) continue;
    const S w = ebx[s] + al * (S(2) * xc[s] - xin[s]);
    const S pb = w - al * clampv(w * ia, lo[s], hi[s]);
    const S rex = ebx[s] - pb, rx = xin[s] - xc[s];
    at<S, IX>(eout, e3 + lane + T * s) = pb;
    st.row((double)rex, (double)rx, (double)ia);
    at<S, IX>(eout, e3 + nx + lane + T * s) = oq[s];
    const S req = eq[s] - oq[s];
    st.row((double)req, (double)(sqn[s] * rx), (double)ia);
    st.col((double)rx, (double)(rex + sqn[s] * req), (double)ia);
  }
  if (lane == 0) {
    const S rs = sv - svp;
    at<S, IX>(eout, e3 + 2 * nx) = osa;
    at<S, IX>(eout, e3 + 2 * nx + 1) = osb;
    const S rea = ea - osa, reb = ebb - osb;
    st.row((double)rea, 0.5 * (double)rs, (double)ia);
    st.row((double)reb, 0.5 * (double)rs, (double)ia);
    st.col((double)rs, 0.5 * ((double)rea + (double)reb), (double)ia);
  }
}

// M d = (d_z - alpha L* d_eta, d_eta - alpha L d_z), the metric of the
// SuperMann line search (Alg. 3): one team of T lanes per family writes the
// family's columns of L* (y^i, s^i, x^i, u^i, tau^c, and x^c, s^c of leaf
// children) and its rows of L (groups 1, 2 of its children, 3 of its leaf
// children), so every entry of M d is written once.
template <typename S, int T>
__device__ __forceinline__ void fam_apply_M(const DevProb<S>& P, const S* __restrict__ d, S* __restrict__ Md, int i,
                                            int lane) {
  const Off<S> O(P);
  const int nx = P.nx, nu = P.nu, fc = P.fc[i], n = P.nch[i];
  const S al = P.alpha;
  const S* dz = d;
  const S* de = d + P.nz;
  S* mz = Md;
  S* me = Md + P.nz;
  const long long zb = O.z2(i), e1 = O.e1(i);
  const S es = de[O.e1s(i)];
  // columns y^i and s^i of L*; rows y and s - b'y of group 1
  double by = 0;
  for (int k = lane; k < 2 * n + 1; k += T) {
    const S bk = (k < n) ? P.p[fc + k] : ((k == 2 * n) ? S(1) : S(0));
    const S yk = dz[zb + k];
    mz[zb + k] = yk - al * (de[e1 + k] - bk * es);
    me[e1 + k] = de[e1 + k] - al * yk;
    by += (double)(bk * yk);
  }
  const S bys = (S)team_sum<T>(by);
  if (lane == 0) {
    mz[O.s(i)] = dz[O.s(i)] - al * es;
    me[O.e1s(i)] = es - al * (dz[O.s(i)] - bys);
  }
  // columns x^i, u^i; rows x, u of group 1 and of the children's group 2
  for (int o = lane; o < nx; o += T) {
    const S xo = dz[O.x(i) + o];
    S acc = de[O.e1x(i) + o];
    for (int k = 0; k < n; ++k) {
      const int c = fc + k;
      const S sq = P.sq[(size_t)c * nx + o];
      const long long e2 = O.e2(c) + o;
      acc += sq * de[e2];
      me[e2] = de[e2] - al * sq * xo;
    }
    mz[O.x(i) + o] = xo - al * acc;
    me[O.e1x(i) + o] = de[O.e1x(i) + o] - al * xo;
  }
  for (int o = lane; o < nu; o += T) {
    const S uo = dz[O.u(i) + o];
    S acc = de[O.e1u(i) + o];
    for (int k = 0; k < n; ++k) {
      const int c = fc + k;
      const S sr = P.sr[(size_t)c * nu + o];
      const long long e2 = O.e2(c) + nx + o;
      acc += sr * de[e2];
      me[e2] = de[e2] - al * sr * uo;
    }
    mz[O.u(i) + o] = uo - al * acc;
    me[O.e1u(i) + o] = de[O.e1u(i) + o] - al * uo;
  }
  // tau^c and the two scalars of group 2
  for (int k = lane; k < n; k += T) {
    const int c = fc + k;
    const long long e2 = O.e2(c) + nx + nu;
    const S tc = dz[O.tau(c)];
    mz[O.tau(c)] = tc - al * S(0.5) * (de[e2] + de[e2 + 1]);
    me[e2] = de[e2] - al * S(0.5) * tc;
    me[e2 + 1] = de[e2 + 1] - al * S(0.5) * tc;
  }
  if (fc < P.nl) return;
  // leaf children: columns x^c, s^c; rows of group 3
  for (int k = 0; k < n; ++k) {
    const int c = fc + k;
    const long long e3 = O.e3(c);
    for (int o = lane; o < nx; o += T) {
      const S xc = dz[O.x(c) + o];
      const S sqn = P.sqN[(size_t)c * nx + o];
      mz[O.x(c) + o] = xc - al * (de[e3 + o] + sqn * de[e3 + nx + o]);
      me[e3 + o] = de[e3 + o] - al * xc;
      me[e3 + nx + o] = de[e3 + nx + o] - al * sqn * xc;
    }
    if (lane == 0) {
      const S sc = dz[O.s(c)];
      mz[O.s(c)] = sc - al * S(0.5) * (de[e3 + 2 * nx] + de[e3 + 2 * nx + 1]);
      me[e3 + 2 * nx] = de[e3 + 2 * nx] - al * S(0.5) * sc;
      me[e3 + 2 * nx + 1] = de[e3 + 2 * nx + 1] - al * S(0.5) * sc;
    }
  }
}

// Anderson step on the device (section 6.2, type-II; one thread, k <= 4):
// the Gram row of the newest difference and the right-hand side <dR_j, r>
// come from the push dot products; the oldest columns are dropped until the
// Gram matrix of the kept ones has lambda_min / lambda_max >= 1e-12 (the
// singular-value ratio 1e-6 of the residual differences; cyclic Jacobi until
// the test is decided) and a Cholesky factor; gamma solves G gamma = rhs. gamma
// is written for every column of the order (0 for dropped ones), and the
// device ring takes the new order (the kept columns) and the direction's
// columns.
// Fixed-size (N <= 4) helpers, fully unrolled so that the matrices stay in
// registers.
template <int N>
__device__ __forceinline__ bool dev_chol(double (&A)[16]) {
#pragma unroll
  for (int j = 0; j < N; ++j) {
    double d = A[j * 4 + j];
#pragma unroll
    for (int k = 0; k < j; ++k) d -= A[j * 4 + k] * A[j * 4 + k];
    if (!(d > 0.0) || !isfinite(d)) return false;
    d = sqrt(d);
    A[j * 4 + j] = d;
#pragma unroll
    for (int i = j + 1; i < N; ++i) {
      double s = A[i * 4 + j];
#pragma unroll
      for (int k = 0; k < j; ++k) s -= A[i * 4 + k] * A[j * 4 + k];
      A[i * 4 + j] = s / d;
    }
  }
  return true;
}

// Rank test of a symmetric N x N matrix: lambda_min / lambda_max >= 1e-12
// with lambda_max > 0. Cyclic Jacobi sweeps until the test is decided: with
// off the sum of squares of the upper off-diagonal entries, every eigenvalue
// lies within e = sqrt(2 off) of a diagonal entry (Weyl), so the extreme
// eigenvalues are within e of the smallest and largest diagonal entries.
template <int N>
__device__ __forceinline__ bool dev_rank_ok(double (&A)[16]) {
  constexpr double kTol = 1e-12;
  for (int sweep = 0;; ++sweep) {
    double off = 0, dmin = A[0], dmax = A[0];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      dmin = fmin(dmin, A[i * 4 + i]);
      dmax = fmax(dmax, A[i * 4 + i]);
#pragma unroll
      for (int j = i + 1; j < N; ++j) off += A[i * 4 + j] * A[i * 4 + j];
    }
    const double e = sqrt(2.0 * off);
    if (dmax - e > 0.0 && dmin - e >= kTol * (dmax + e)) return true;           // certainly passes
    if (dmax + e <= 0.0 || (dmax - e > 0.0 && dmin + e < kTol * (dmax - e))) return false;  // certainly fails
    if (sweep == 60 || off < 1e-300) return dmax > 0.0 && dmin >= kTol * dmax;  // the diagonal is the spectrum
#pragma unroll
    for (int p = 0; p < N; ++p)
#pragma unroll
      for (int q = p + 1; q < N; ++q) {
        const double apq = A[p * 4 + q];
        if (apq != 0.0) {
          const double th = 0.5 * (A[q * 4 + q] - A[p * 4 + p]) / apq;
          const double t = (th >= 0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
          const double c = 1.0 / sqrt(t * t + 1.0), s = t * c;
#pragma unroll
          for (int k = 0; k < N; ++k) {
            const double akp = A[k * 4 + p], akq = A[k * 4 + q];
            A[k * 4 + p] = c * akp - s * akq;
            A[k * 4 + q] = s * akp + c * akq;
          }
#pragma unroll
          for (int k = 0; k < N; ++k) {
            const double apk = A[p * 4 + k], aqk = A[q * 4 + k];
            A[p * 4 + k] = c * apk - s * aqk;
            A[q * 4 + k] = s * apk + c * aqk;
          }
        }
      }
  }
}

// Rank test and solve for the last N of the k active columns (rows/cols
// `off..off+N` of Gk, right-hand side rk); true when kept.
template <int N, int off>
__device__ __forceinline__ bool dev_aa_try(const double (&Gk)[16], const double (&rk)[4], double (&g)[4]) {
  double E[16], L[16];
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < N; ++j) E[i * 4 + j] = L[i * 4 + j] = Gk[(off + i) * 4 + off + j];
  if (!dev_rank_ok<N>(E) || !dev_chol<N>(L)) return false;
  double y[4];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    double s = rk[off + i];
#pragma unroll
    for (int j = 0; j < i; ++j) s -= L[i * 4 + j] * y[j];
    y[i] = s / L[i * 4 + i];
  }
#pragma unroll
  for (int i = N - 1; i >= 0; --i) {
    double s = y[i];
#pragma unroll
    for (int j = i + 1; j < N; ++j) s -= L[j * 4 + i] * g[off + j];
    g[off + i] = s / L[i * 4 + i];
  }
  return true;
}

// Tries the last K - DROP columns, then fewer; the number kept (0: none).
template <int K, int DROP>
__device__ __forceinline__ int aa_try_from(const double (&Gk)[16], const double (&rk)[4], double (&g)[4]) {
  if constexpr (DROP >= K) {
    return 0;
  } else {
    if (dev_aa_try<K - DROP, DROP>(Gk, rk, g)) return K - DROP;
    return aa_try_from<K, DROP + 1>(Gk, rk, g);
  }
}

// MO columns before the push (all indices fixed at compile time). Gold:
// the Gram entries of the old columns (oldest first), read before the sums
// were done; the new column's entries and the right-hand side <dR_j, r>
// come from the dots. The new row is stored in G (by slot) for later pushes.
template <int MO>
__device__ __forceinline__ void aa_solve_dev(double* __restrict__ G, const double (&dots)[8],
                                             const double (&Gold)[16], const AAPush& a,
                                             double* __restrict__ gamma, AARingDev* __restrict__ ring) {
  const int m = a.m, slot = a.slot;
#pragma unroll
  for (int j = 0; j < MO; ++j) {
    G[a.order_old[j] * m + slot] = dots[j];
    G[slot * m + a.order_old[j]] = dots[j];
  }
  G[slot * m + slot] = dots[MO];
  constexpr int k = MO + 1;  // order_new = order_old + [slot]
  // Gram matrix and right-hand side of the active columns, in registers
  double Gk[16], rk[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    rk[i] = i < MO ? dots[MO + 1 + i] : (i == MO ? dots[2 * MO + 1] : 0.0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      Gk[i * 4 + j] = (i < MO && j < MO) ? Gold[i * 4 + j]
                    : (i == MO && j < MO) ? dots[j]
                    : (j == MO && i < MO) ? dots[i]
                    : (i == MO && j == MO) ? dots[MO] : 0.0;
  }
  double g[4] = {0, 0, 0, 0};
  // drop the oldest columns until the rest pass the rank test
  const int kept = aa_try_from<k, 0>(Gk, rk, g);
  if (kept == 0) g[0] = g[1] = g[2] = g[3] = 0.0;
#pragma unroll
  for (int j = 0; j < k; ++j) gamma[j] = g[j];
  // the ring: the direction uses the k columns (dropped ones with gamma 0);
  // the next push keeps the newest `kept`
  int ord[4] = {0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < MO; ++j) ord[j] = a.order_old[j];
  ord[MO] = slot;
  ring->dk = k;
#pragma unroll
  for (int j = 0; j < k; ++j) ring->dslot[j] = ord[j];
  ring->cnt = kept;
#pragma unroll
  for (int j = 0; j < k; ++j) {
    int sel = 0;
#pragma unroll
    for (int q = 0; q < k; ++q) sel = (q == k - kept + j) ? ord[q] : sel;
    if (j < kept) ring->order[j] = sel;
  }
}

// The push that follows the ring as the last solve left it: the new column
// takes the oldest slot when the ring is full, else the lowest free one; the
// dots run against the other columns of the order.
__device__ __forceinline__ AAPush aa_next_push(const AARingDev* ring) {
  // (fixed indices and selects only, so that nothing lands in scratch)
  AAPush a{};
  a.m = ring->m;
  const int cnt = ring->cnt;
  int o[kAAMax];
#pragma unroll
  for (int j = 0; j < kAAMax; ++j) o[j] = ring->order[j];
  const bool full = cnt == a.m;
  a.mo = full ? cnt - 1 : cnt;
#pragma unroll
  for (int j = 0; j < kAAMax; ++j) a.order_old[j] = full ? (j + 1 < kAAMax ? o[j + 1] : 0) : o[j];
  int fr = kAAMax;  // lowest slot not in the order
#pragma unroll
  for (int s = kAAMax - 1; s >= 0; --s) {
    bool used = false;
#pragma unroll
    for (int j = 0; j < kAAMax; ++j) used = used || (j < cnt && o[j] == s);
    if (!used && s < a.m) fr = s;
  }
  a.slot = full ? o[0] : fr;
  return a;
}

// Sweep buffers of a shared-tree batch hold kTileCols instances of an entry side
// by side: entry e of instance b at tile_base(b, entries per instance) +
// e * kTileCols.
constexpr int kTileCols = 16;
__device__ __forceinline__ size_t tile_base(size_t b, size_t per) {
  return b / kTileCols * per * kTileCols + b % kTileCols;
}

// Tagged words: element e of a vector occupies kTW<S> 64-bit words, each
// holding (epoch << 32) | one 32-bit half of the value.
template <typename S>
constexpr int kTW = sizeof(S) / 4;

template <typename S>
__device__ __forceinline__ void put_tagged(unsigned long long* p, S v, unsigned tag) {
  unsigned h[kTW<S>];
  __builtin_memcpy(h, &v, sizeof(S));
  const unsigned long long hi = (unsigned long long)tag << 32;
#pragma unroll
  for (int k = 0; k < kTW<S>; ++k) __hip_atomic_store(p + k, hi | h[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename S>
__device__ __forceinline__ bool get_tagged(const unsigned long long* p, unsigned tag, S& v) {
  unsigned h[kTW<S>];
  bool ok = true;
#pragma unroll
  for (int k = 0; k < kTW<S>; ++k) {
    const unsigned long long w = __hip_atomic_load(p + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ok = ok && (unsigned)(w >> 32) == tag;
    h[k] = (unsigned)w;
  }
  __builtin_memcpy(&v, h, sizeof(S));
  return ok;
}

}  // namespace spk
