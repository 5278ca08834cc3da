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

// Transpose of the root-state map Phi of the S1 projection, one stage per
// launch (stage N-1 .. 0) for every instance: mu^j = c_x^j at leaves, mu^i =
// c_x^i + K^i' c_u^i + sum_c Abar^c' mu^c; mu^0 is the gradient with respect
// to x0, written to gx0. One wavefront per (node, instance), lane o on
// component o (nx <= 64): the rows of K and Abar are read coalesced and the
// sums run in the order of the formula. Bound by the latency of a stage's
// chain; one thread per node walked nx (nu + n nx) dependent loads (85 us per
// stage on the 95-node tree in FP64, once per instance: 43 of the 60 ms of a
// 64-instance adjoint of 32 applications, now 10.5 ms in all).
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

__global__ void k_copy_elem_d(double* dst, const double* src) { dst[0] = src[0]; }
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
