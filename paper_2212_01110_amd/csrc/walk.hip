// Walk form of the two Alg. 2 sweeps: like the dataflow form (flow.hip), both
// sweeps of one evaluation of T in one persistent launch whose workgroups
// pass q, d and x as tagged words, for trees in which the dependent stages
// and not the bytes set the time.
//
// There, a stage costs what the next one waits for: the value's way through
// memory (about 0.6 us) and one mat-vec phase. Two things make this short:
//   - The weights wait for the vector, not the other way round: an item's
//     matrices are copied into LDS and from there into registers before its
//     vector is polled, and the products take a register, a scalar and one
//     instruction each (mat-vec phase below).
//   - Runs of stages stay in one workgroup, all their matrices in LDS before
//     the run's first value arrives, so no value passes through memory inside
//     a run. A backward item goes on from its family to the parents for as
//     long as they have one child (a chain). A forward item is a piece of a
//     path, from a node down to one of its descendants some stages below;
//     pieces recompute the states that they share, and the first piece through
//     a node writes them. Stages where the pieces would be too many, or too
//     long for the LDS, have items as in the dataflow form: chunks of (at most
//     nc) children of a family; a chunk of the backward sweep that is not its
//     family's last publishes its partial sums, which the last one adds.
// Sweeps in the dataflow form and here: 15 nodes (n_x 3, n_u 2, FP64) 15.0 and
// 8.2 us; 95 nodes (n_x 20, n_u 10, FP64) 35.3 and 18.0; 223 nodes (the same)
// 44.2 and 21.3; 2047 nodes (n_x = n_u = 20, FP32) 53 and 26; 4095 nodes
// (n_x = n_u = 50, FP32) 101 and 64. A branching stage is now 1.2 us, half of
// it the values' way through memory; a stage inside a run 0.5 us.
//
// Items wait only on items with a smaller index, and a workgroup runs its own
// in increasing order (b, b + G, ..., G the resident capacity), so the launch
// drains; every poll is bounded, as in the dataflow form.
#include "flow_common.h"

#include <algorithm>

namespace spk {

namespace {

// Word offsets of the dynamic LDS regions (32-bit words; every region starts at
// a multiple of 64 words, so that the copies' 16-byte units land aligned).
struct WalkLds {
  int esz;     // words per element
  int sA, sB;  // per-child strides of the At / Abar and Bt / B regions
  int oA, oB, oR, oK, oQ, oX, oU, oRed;  // oK: P1 (backward) or K (forward)
  int nc;      // children per chunk
  int sRed;    // the partial sums of 4 wavefronts, n_x + n_u outputs each
  int words;
  __host__ __device__ static int pad(int w) { return (w + 63) & ~63; }
  __host__ __device__ WalkLds(int nx, int nu, int nc_, int esz_) {
    esz = esz_;
    nc = nc_;
    sA = pad(nx * nx * esz);
    sB = pad(nx * nu * esz);
    oA = 0;
    oB = oA + nc * sA;
    oR = oB + nc * sB;
    oK = oR + pad(nu * nu * esz);
    oQ = oK + pad(nx * nu * esz);  // children's q (chunk), row stride nx
    oX = oQ + pad(nc * nx * esz);  // xbar (backward) or x (forward)
    oU = oX + pad(nx * esz);       // ubar (backward) or d (forward)
    oRed = oU + pad(nu * esz);
    sRed = 4 * pad((nx + nu) * esz);
    const int fwd = pad(4 * (nc * nx + nu) * esz);
    words = oRed + (fwd > sRed ? fwd : sRed);
  }
  // A chain's further links follow the item's own regions: At, Bt, R~^{-1}, P1,
  // xbar, ubar and the head (P1 ubar - xbar, R~^{-1} ubar).
  __host__ __device__ int chain_link() const { return sA + sB + (oQ - oR) + (oRed - oX) + sRed / 4; }
  // A path piece consists of its links: Abar, B, K and the head (B d, d).
  __host__ __device__ int path_link() const { return sA + sB + (oQ - oK) + sRed / 4; }
};

// ---------------------------------------------------------------- mat-vec phase
// Matrices are input-major (input k's row holds its weights for all outputs).
// Lane l of a wavefront owns outputs l and, with two slots, 64 + l of the
// concatenated outputs of two blocks with the same inputs (backward: q and d;
// forward: the first child's x, and u). A row's input value is the same for
// all lanes of a wavefront: it is taken from the lane that holds it into a
// scalar register, and the weights go to registers before it is there.
// An item's first stage has its rows on the four wavefronts in turn (w, w + 4,
// ...), whose partial sums meet in LDS. The stages of a chain or path after it
// run on one wavefront alone: outputs and inputs are in the same lanes, so
// that a stage is n_x multiply-adds and nothing else, where four wavefronts
// have a barrier and two trips through LDS each (n_x 20, n_u 10, FP64: 0.5 us a
// stage against 0.65 to 1.0).
//
// R: rows per wavefront (at least a quarter of either dimension); SL: slots
// (two where n_x + n_u exceeds 64).
// Values that the item loop would otherwise keep (with every pointer and
// mask derived from them) in more scalar registers than there are.
__device__ __forceinline__ int here_s(int v) {
  asm volatile("" : "+s"(v));
  return v;
}
__device__ __forceinline__ int here_v(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
template <typename S>
__device__ __forceinline__ S lane_val(S v, int k) {
  if constexpr (sizeof(S) == 4) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), k));
  } else {
    const long long b = __builtin_bit_cast(long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, k);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), k);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
  }
}

// The outputs of this lane in two blocks of n1 and n2 outputs: position in the
// block and row stride per slot (lanes past the outputs repeat output 0).
template <int SL>
struct LaneOut {
  int pos[SL], st[SL];
  bool second[SL];
  __device__ __forceinline__ LaneOut(int n1, int n2, int lane) {
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      const int o = lane + 64 * s;
      second[s] = o >= n1 && o < n1 + n2;
      pos[s] = o < n1 ? o : second[s] ? o - n1 : 0;
      st[s] = second[s] ? n2 : n1;
    }
  }
};

// Weights of rows w, w + 4, ... (the last of the n rows again past the end)
// of the blocks at elements b1 and b2.
template <typename S, int R, int SL>
__device__ __forceinline__ void load_rows(const S* M, int b1, int b2, const LaneOut<SL>& O, int n, int w,
                                          S (&m)[SL][R]) {
#pragma unroll
  for (int s = 0; s < SL; ++s) {
    const int b = (O.second[s] ? b2 : b1) + O.pos[s];
#pragma unroll
    for (int r = 0; r < R; ++r) m[s][r] = M[b + __umul24(min(w + 4 * r, n - 1), O.st[s])];
  }
}

// a += their products with vector v (lane k holds entry k, zero past the end)
template <typename S, int R, int SL>
__device__ __forceinline__ void fma_rows(const S (&m)[SL][R], S v, int w, S (&a)[SL][2]) {
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const S vk = lane_val<S>(v, w + 4 * r);
#pragma unroll
    for (int s = 0; s < SL; ++s) a[s][r & 1] += m[s][r] * vk;
  }
}

// On one wavefront alone, rows go kCh<R, SL> at a time (4 R is a multiple).
template <int R, int SL>
constexpr int kCh = SL > 1 ? 4 : R == 2 ? 8 : R == 3 ? 6 : R == 5 ? 10 : R == 13 ? 13 : 8;

// Weights of rows k0, k0 + 1, ... (the last again past the end).
template <typename S, int CH, int SL>
__device__ __forceinline__ void load_run(const S* M, int b1, int b2, const LaneOut<SL>& O, int n, int k0,
                                         S (&m)[SL][CH]) {
#pragma unroll
  for (int s = 0; s < SL; ++s) {
    const int b = (O.second[s] ? b2 : b1) + O.pos[s];
#pragma unroll
    for (int r = 0; r < CH; ++r) m[s][r] = M[b + __umul24(min(k0 + r, n - 1), O.st[s])];
  }
}

template <typename S, int CH, int SL>
__device__ __forceinline__ void fma_run(const S (&m)[SL][CH], S v, int k0, S (&a)[SL][2]) {
#pragma unroll
  for (int r = 0; r < CH; ++r) {
    const S vk = lane_val<S>(v, k0 + r);
#pragma unroll
    for (int s = 0; s < SL; ++s) a[s][r & 1] += m[s][r] * vk;
  }
}

// All n rows of one pair of blocks on one wavefront.
template <typename S, int R, int SL>
__device__ __forceinline__ void sum_rows(const S* M, int b1, int b2, const LaneOut<SL>& O, int n, S v,
                                         S (&a)[SL][2]) {
  constexpr int CH = kCh<R, SL>;
  S m[SL][CH];
#pragma unroll 1
  for (int k0 = 0; k0 < n; k0 += CH) {
    load_run<S, CH, SL>(M, b1, b2, O, n, k0, m);
    fma_run<S, CH, SL>(m, v, k0, a);
  }
}

// Stages [l0, l1) of a run on one wavefront: v = the products of link l's
// blocks (elements at(l) and at(l) + off2) with v, plus its head (element
// head(l)); done(l, outputs) takes the outputs of each slot, of which lanes
// below n hold the next v. Weights are read one chunk of rows ahead, across
// links too (a link's first chunk has registers of its own).
template <typename S, int R, int SL, typename At, typename Head, typename Done>
__device__ __forceinline__ void run_links(const S* M, const LaneOut<SL>& O, int n, int nout, int off2, int lane, int l0,
                                          int l1, S v, At at, Head head, Done done) {
  constexpr int CH = kCh<R, SL>, NC = 4 * R / CH;
  if (l0 >= l1) return;
  S m0[SL][CH], mx[2][SL][CH], h[SL];
  auto heads = [&](int l) {
#pragma unroll
    for (int s = 0; s < SL; ++s) h[s] = M[head(l) + min(lane + 64 * s, nout - 1)];
  };
  heads(l0);
  load_run<S, CH, SL>(M, at(l0), at(l0) + off2, O, n, 0, m0);
#pragma unroll 1
  for (int l = l0; l < l1; ++l) {
    const int b = at(l), bn = at(min(l + 1, l1 - 1));
    S a[SL][2] = {};
    if (CH < n) load_run<S, CH, SL>(M, b, b + off2, O, n, CH, mx[0]);
    fma_run<S, CH, SL>(m0, v, 0, a);
    load_run<S, CH, SL>(M, bn, bn + off2, O, n, 0, m0);
#pragma unroll
    for (int c = 1; c < NC; ++c)
      if (c * CH < n) {
        if (c + 1 < NC && (c + 1) * CH < n) load_run<S, CH, SL>(M, b, b + off2, O, n, (c + 1) * CH, mx[c & 1]);
        fma_run<S, CH, SL>(mx[(c - 1) & 1], v, c * CH, a);
      }
    S o[SL];
#pragma unroll
    for (int s = 0; s < SL; ++s) o[s] = (a[s][0] + a[s][1]) + h[s];
    v = lane < n ? o[0] : S(0);
    heads(min(l + 1, l1 - 1));
    done(l, o);
  }
}

// This wavefront's partial sums of the nout outputs, and an output's sum over
// the wavefronts (stride elements from one to the next).
template <typename S, int SL>
__device__ __forceinline__ void put_part(S* red, int nout, int lane, const S (&a)[SL][2]) {
#pragma unroll
  for (int s = 0; s < SL; ++s)
    if (lane + 64 * s < nout) red[lane + 64 * s] = a[s][0] + a[s][1];
}

template <typename S>
__device__ __forceinline__ S fold4(const S* red, int stride, int o) {
  const S p0 = red[o], p1 = red[stride + o], p2 = red[2 * stride + o], p3 = red[3 * stride + o];
  return (p0 + p1) + (p2 + p3);
}

template <typename S>
struct WalkArgs {
  DevProb<S> P;
  S* zout;
  const double* x0;
  const S* xbar;
  const S* ubar;
  const S* seeds;            // q of the leaf children (pre-pass), plain
  unsigned long long* qt;    // [nl][nx] tagged q
  unsigned long long* dt;    // [nl][nu] tagged d
  unsigned long long* xt;    // [nn][nx] tagged x (forward step of the parent)
  unsigned long long* pt;    // [slots][nx + nu] tagged partial sums of backward chunks
  const int* items;          // records of rs ints (WalkPlan): backward items, then forward
  const int* pbase;          // [nl] first partial slot of a family with several chunks
  unsigned* err;             // [1]
  unsigned tag;
  unsigned spin;             // polls of one bounded wait before it gives up
  int nc, nbwd, nitems, rs;
};

// Entry k of the record that lane k holds (the same in every lane).
__device__ __forceinline__ int rec_int(int rv, int k) { return __builtin_amdgcn_readlane(rv, k); }

// The launch's arguments, read where they are used (scalar loads).
template <typename S>
using Args = const __attribute__((address_space(4))) WalkArgs<S>*;
template <typename S>
__device__ __forceinline__ Args<S> here_args() {
  auto p = reinterpret_cast<unsigned long long>(__builtin_amdgcn_kernarg_segment_ptr());
  asm volatile("" : "+s"(p));
  return reinterpret_cast<Args<S>>(p);
}

// Copies nwords 32-bit words from global memory into LDS (dst = word offset, a
// multiple of 64) by the calling wavefront: 16 bytes per lane from an aligned
// source, and 4 bytes per lane for what is left (all of it from another).
__device__ __forceinline__ void copy_in(const void* src, unsigned* lds, int dst, int nwords, int lane) {
  const char* s = static_cast<const char*>(src);
  int done = 0;
  if ((reinterpret_cast<uintptr_t>(src) & 15u) == 0) {
    const int units = nwords >> 2;
    for (int u = 0; u < units; u += 64)
      if (u + lane < units)
        __builtin_amdgcn_global_load_lds(s + (unsigned)((u + lane) * 16), (lds_void*)(lds + dst + u * 4), 16, 0, 0);
    done = units << 2;
  }
  for (int e = done; e < nwords; e += 64)
    if (e + lane < nwords)
      __builtin_amdgcn_global_load_lds(s + (unsigned)((e + lane) * 4), (lds_void*)(lds + dst + e), 4, 0, 0);
}

// One wavefront's lanes below n <= 64 poll an element each of two vectors (one
// memory round trip for both) until all carry tag (bounded); lanes past the
// end hold zero.
template <typename S>
__device__ __forceinline__ void wait_lanes(const unsigned long long* src0, const unsigned long long* src1, int n,
                                           int lane, unsigned tag, unsigned* err, unsigned spin, S& v0, S& v1) {
  const unsigned e = (unsigned)(lane < n ? lane : 0) * kTW<S>;
  const S zero = 0;
  for (unsigned it = 0; it < spin; ++it) {
    const bool ok0 = get_tagged<S>(src0 + e, tag, v0), ok1 = get_tagged<S>(src1 + e, tag, v1);
    const bool done = __all(ok0 && ok1);
    v0 = lane < n ? v0 : zero;
    v1 = lane < n ? v1 : zero;
    if (done) return;
    if ((it & 255u) == 255u && ld_flag(err) != 0u) return;
    __builtin_amdgcn_s_sleep(1);
  }
  v0 = v1 = 0;
  __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The same for one vector.
template <typename S>
__device__ __forceinline__ S wait_lane(const unsigned long long* src, int n, int lane, unsigned tag, unsigned* err,
                                       unsigned spin) {
  S v0, v1;
  wait_lanes<S>(src, src, n, lane, tag, err, spin, v0, v1);
  return v0;
}

// Sum, in slot order, of entry e of the first n partial records at pp (stride
// rs elements), polled by the calling thread until every word carries tag
// (bounded).
template <typename S>
__device__ __forceinline__ S sum_partials(const unsigned long long* pp, int n, int rs, int e, unsigned tag,
                                          unsigned* err, unsigned spin) {
  for (unsigned it = 0; it < spin; ++it) {
    bool ok = true;
    S a = 0;
    for (int q = 0; q < n; ++q) {
      S v;
      ok = get_tagged<S>(pp + ((size_t)q * rs + e) * kTW<S>, tag, v) && ok;
      a += v;
    }
    if (ok) return a;
    if ((it & 255u) == 255u && ld_flag(err) != 0u) return 0;
    __builtin_amdgcn_s_sleep(1);
  }
  __hip_atomic_store(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return 0;
}

// ---------------------------------------------------------------- backward item
// Alg. 2 backward step in one mat-vec phase: substituting
// g = ubar - sum_c B^c' q^c into d = R~^{-1} g and q = M1 g - K' ubar - xbar
// + sum_c Abar^c' q^c (M1 = (K' + W) R~^{-1}) gives
//   d = R~^{-1} ubar + sum_c Bt^c q^c,   q = P1 ubar - xbar + sum_c At^c q^c
// with Bt^c = -R~^{-1} B^c', At^c = Abar^c' - M1 B^c', P1 = M1 - K' formed
// offline in FP64 (equal to Alg. 2's step in exact arithmetic).
// Chunk j of family i (children j nc, ...). Wavefront 0 copies the At of the
// children (and of the chain's links), 1 the Bt, 2 P1 and xbar, 3 R~^{-1} and
// ubar, and the seeds of leaf children; all poll the children's q. A chunk that is not the family's last
// publishes its partial sums; the last chunk adds P1 ubar and R~^{-1} ubar and
// the earlier chunks' partial sums (chunk order) and publishes d and q, or with
// a chain goes on with q to the parent, on wavefront 0.
template <typename S, int R, int SL>
__device__ __forceinline__ void walk_bwd(unsigned* lds, int rv) {
  constexpr int NH = kTW<S> * SL * R <= 32 ? 2 : 1;  // children whose weights are held
  const Args<S> A = here_args<S>();
  const int t = here_v(threadIdx.x), w = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  const int code = rec_int(rv, 0), m = rec_int(rv, 1), fc = rec_int(rv, 2), n = rec_int(rv, 3);
  const int i = code / kChunkCodes, j = code % kChunkCodes;
  const int nx = here_s(A->P.nx), nu = here_s(A->P.nu), nout = nx + nu;
  const WalkLds L(nx, nu, A->nc, (int)(sizeof(S) / 4));
  constexpr int es = sizeof(S) / 4;
  const S* M = reinterpret_cast<const S*>(lds);
  const S* qv = reinterpret_cast<const S*>(lds + L.oQ);
  S* red = reinterpret_cast<S*>(lds + L.oRed);
  const bool leafkids = fc >= A->P.nl;
  const int k0 = j * L.nc, kc = min(L.nc, n - k0);
  const bool last = k0 + kc == n;
  // link l >= 1 from word cb + l LW: At, Bt, R~^{-1}, P1, xbar, ubar, head
  const int LW = L.chain_link(), cb = L.words - LW, cR = L.sA + L.sB, cK = cR + (L.oK - L.oR), cX = cR + (L.oQ - L.oR),
            cU = cX + (L.oU - L.oX), cH = cX + (L.oRed - L.oX);
  {
    const S* mat = w == 0 ? A->P.AtR : w == 1 ? A->P.BtR : w == 2 ? A->P.P1C : A->P.Rinv;
    const int len = (w == 3 ? nu : nx) * (w == 0 ? nx : nu);
    const int off = w == 0 ? 0 : w == 1 ? L.sA : w == 2 ? cK : cR;  // within a link
    const S* vec = w == 2 ? A->xbar : A->ubar;
    const int vlen = w == 2 ? nx : nu, voff = w == 2 ? cX : cU;
    if (w < 2) {
      for (int k = 0; k < kc; ++k)
        copy_in(mat + (size_t)(fc + k0 + k) * len, lds, w == 0 ? L.oA + k * L.sA : L.oB + k * L.sB, len * es, lane);
    } else if (last) {
      copy_in(mat + (size_t)i * len, lds, w == 2 ? L.oK : L.oR, len * es, lane);
      copy_in(vec + (size_t)i * vlen, lds, w == 2 ? L.oX : L.oU, vlen * es, lane);
    }
    if (leafkids && w == 3)  // seeds -xbar of the leaf children, written by the pre-pass
      copy_in(A->seeds + (size_t)(fc + k0) * nx, lds, L.oQ, kc * nx * es, lane);
    for (int l = 1, c = i; l < m; ++l) {
      const int f = rec_int(rv, 3 + l), o = cb + l * LW;
      copy_in(mat + (size_t)(w < 2 ? c : f) * len, lds, o + off, len * es, lane);
      if (w >= 2) copy_in(vec + (size_t)f * vlen, lds, o + voff, vlen * es, lane);
      c = f;
    }
  }
  wait_vm();
  __syncthreads();
  const LaneOut<SL> O(nx, nu, lane);
  S a[SL][2] = {}, mr[NH][SL][R];
  // what does not wait for q: the heads of the chain's links, a wavefront each,
  // and the family's own products with ubar
  for (int l = 1 + w; l < m; l += 4) {
    const int o = cb + l * LW;
    const S* ub = reinterpret_cast<const S*>(lds + o + cU);
    const S* xb = reinterpret_cast<const S*>(lds + o + cX);
    S b[SL][2] = {};
    sum_rows<S, R, SL>(M, (o + cK) / es, (o + cR) / es, O, nu, lane < nu ? ub[lane] : S(0), b);
    if (lane < nx) b[0][0] -= xb[lane];
    put_part<S, SL>(reinterpret_cast<S*>(lds + o + cH), nout, lane, b);
  }
  if (last) {
    const S* ub = reinterpret_cast<const S*>(lds + L.oU);
    load_rows<S, R, SL>(M, L.oK / es, L.oR / es, O, nu, w, mr[0]);
    fma_rows<S, R, SL>(mr[0], lane < nu ? ub[lane] : S(0), w, a);
  }
#pragma unroll
  for (int h = 0; h < NH; ++h)
    if (h < kc) load_rows<S, R, SL>(M, (L.oA + h * L.sA) / es, (L.oB + h * L.sB) / es, O, nx, w, mr[h]);
  // children's q, two at a time: the seeds in LDS, or from their backward items
  // (every wavefront polls for itself: no trip through LDS and no barrier)
  const unsigned long long* const qc = A->qt + (size_t)(fc + k0) * nx * kTW<S>;
  for (int k = 0; k < kc; k += 2) {
    const int k1 = min(k + 1, kc - 1);
    S q0, q1;
    if (leafkids) {
      q0 = lane < nx ? qv[k * nx + lane] : S(0);
      q1 = lane < nx ? qv[k1 * nx + lane] : S(0);
    } else {
      wait_lanes<S>(qc + (size_t)k * nx * kTW<S>, qc + (size_t)k1 * nx * kTW<S>, nx, lane, A->tag, A->err, A->spin, q0,
                    q1);
    }
    if (k > 0) load_rows<S, R, SL>(M, (L.oA + k * L.sA) / es, (L.oB + k * L.sB) / es, O, nx, w, mr[0]);
    fma_rows<S, R, SL>(mr[0], q0, w, a);
    if (k1 > k) {
      if (k > 0 || NH == 1)
        load_rows<S, R, SL>(M, (L.oA + k1 * L.sA) / es, (L.oB + k1 * L.sB) / es, O, nx, w, mr[NH - 1]);
      fma_rows<S, R, SL>(mr[NH - 1], q1, w, a);
    }
  }
  put_part<S, SL>(red + w * nout, nout, lane, a);
  __syncthreads();
  // outputs lane, 64 + lane: of all wavefronts, one after the other without a
  // chain, of wavefront 0 with one
  const unsigned tag = A->tag;
  unsigned long long* const qt = A->qt;
  unsigned long long* const dt = A->dt;
  auto publish = [&](int f, int o, S v) {
    if (o < nx)
      put_tagged<S>(qt + ((size_t)f * nx + o) * kTW<S>, v, tag);
    else
      put_tagged<S>(dt + ((size_t)f * nu + (o - nx)) * kTW<S>, v, tag);
  };
  const int nprev = k0 / L.nc;
  if (!last || m == 1) {
    if (t < nout) {
      S v = fold4<S>(red, nout, t);
      if (!last) {
        put_tagged<S>(A->pt + ((size_t)(A->pbase[i] + j) * nout + t) * kTW<S>, v, tag);
      } else {
        if (nprev > 0)
          v += sum_partials<S>(A->pt + (size_t)A->pbase[i] * nout * kTW<S>, nprev, nout, t, tag, A->err, A->spin);
        if (t < nx) v -= reinterpret_cast<const S*>(lds + L.oX)[t];
        publish(i, t, v);
      }
    }
  } else if (w == 0) {
    S q = 0;
#pragma unroll
    for (int s = 0; s < SL; ++s) {
      const int o = lane + 64 * s;
      if (o < nout) {
        S v = fold4<S>(red, nout, o);
        if (nprev > 0)
          v += sum_partials<S>(A->pt + (size_t)A->pbase[i] * nout * kTW<S>, nprev, nout, o, tag, A->err, A->spin);
        if (o < nx)
          q = v - reinterpret_cast<const S*>(lds + L.oX)[o];
        else
          publish(i, o, v);
      }
    }
    run_links<S, R, SL>(
        M, O, nx, nout, L.sA / es, lane, 1, m, q, [&](int l) { return (cb + l * LW) / es; },
        [&](int l) { return (cb + l * LW + cH) / es; },
        [&](int l, const S(&v)[SL]) {
          const int f = rec_int(rv, 3 + l);
#pragma unroll
          for (int s = 0; s < SL; ++s) {
            const int o = lane + 64 * s;
            if (o < nout && (o >= nx || l + 1 == m)) publish(f, o, v[s]);
          }
        });
  }
  __syncthreads();  // LDS reuse by the next item
}

// ---------------------------------------------------------------- forward item
// u = K x + d (chunk 0); x^c = Abar^c x + B^c d for the chunk's children;
// x^0 = x0 at the root. Wavefronts 0 and 3 copy the Abar, 1 the B, 2 K;
// all poll d (the family's backward step, long there below the top stages) and
// then x (the parent's forward step).
template <typename S, int R, int SL>
__device__ __forceinline__ void walk_fwd(unsigned* lds, int rv) {
  constexpr int NH = kTW<S> * R <= 16 ? 2 : 1;  // children whose weights are held
  const Args<S> A = here_args<S>();
  const int t = here_v(threadIdx.x), w = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  const int code = rec_int(rv, 0), i = code / kChunkCodes, j = code % kChunkCodes;
  const int nx = here_s(A->P.nx), nu = here_s(A->P.nu), nl = A->P.nl, fc = rec_int(rv, 2), n = rec_int(rv, 3);
  const WalkLds L(nx, nu, A->nc, (int)(sizeof(S) / 4));
  constexpr int es = sizeof(S) / 4;
  const S* M = reinterpret_cast<const S*>(lds);
  S* red = reinterpret_cast<S*>(lds + L.oRed);
  const int k0 = j * L.nc, kc = min(L.nc, n - k0);
  const int nU = j == 0 ? nu : 0, nout = kc * nx + nU;  // outputs: first child's x, u, the other children's x
  if (w == 2) {
    if (j == 0) copy_in(A->P.KC + (size_t)i * nx * nu, lds, L.oK, nx * nu * es, lane);
  } else {
    const S* mat = w == 1 ? A->P.BC : A->P.AbC;
    const int len = nx * (w == 1 ? nu : nx), o = w == 1 ? L.oB : L.oA, st = w == 1 ? L.sB : L.sA;
    for (int k = w == 3 ? 1 : 0; k < kc; k += w == 1 ? 1 : 2)
      copy_in(mat + (size_t)(fc + k0 + k) * len, lds, o + k * st, len * es, lane);
  }
  wait_vm();
  __syncthreads();
  const LaneOut<SL> O(nx, nU, lane);
  const LaneOut<1> X(nx, 0, lane);
  S m0[SL][R], mb[NH][1][R], m1[1][R];
  load_rows<S, R, SL>(M, L.oA / es, L.oK / es, O, nx, w, m0);
  load_rows<S, R, 1>(M, L.oB / es, 0, X, nu, w, mb[0]);
  if (NH > 1 && kc > 1) {
    load_rows<S, R, 1>(M, (L.oA + L.sA) / es, 0, X, nx, w, m1);
    load_rows<S, R, 1>(M, (L.oB + L.sB) / es, 0, X, nu, w, mb[NH - 1]);
  }
  S* const zout = A->zout;
  S x = 0;
  const S d = wait_lane<S>(A->dt + (size_t)i * nu * kTW<S>, nu, lane, A->tag, A->err, A->spin);
  if (i != 0) {
    x = wait_lane<S>(A->xt + (size_t)i * nx * kTW<S>, nx, lane, A->tag, A->err, A->spin);
  } else if (lane < nx) {
    x = (S)A->x0[lane];
    if (j == 0 && w == 0) zout[1 + lane] = x;
  }
  S* const part = red + w * nout;
  {
    S a[SL][2] = {}, ab[1][2] = {};
    fma_rows<S, R, 1>(mb[0], d, w, ab);
    fma_rows<S, R, SL>(m0, x, w, a);
    if (lane < nx) {
      a[0][0] += ab[0][0];
      a[0][1] += ab[0][1];
    }
    put_part<S, SL>(part, nx + nU, lane, a);
  }
  for (int k = 1; k < kc; ++k) {
    S a[1][2] = {};
    if (NH == 1 || k > 1) {
      load_rows<S, R, 1>(M, (L.oA + k * L.sA) / es, 0, X, nx, w, m1);
      load_rows<S, R, 1>(M, (L.oB + k * L.sB) / es, 0, X, nu, w, mb[NH - 1]);
    }
    fma_rows<S, R, 1>(m1, x, w, a);
    fma_rows<S, R, 1>(mb[NH - 1], d, w, a);
    put_part<S, 1>(part + k * nx + nU, nx, lane, a);
  }
  __syncthreads();
  // wavefront 3: u; the others: the children's x, in turn
  if (w == 3) {
    if (lane < nU) zout[A->P.zU + (long long)i * nu + lane] = fold4<S>(red, nout, nx + lane) + d;
  } else if (lane < nx) {
    unsigned long long* const xt = A->xt;
    const unsigned tag = A->tag;
    for (int k = w; k < kc; k += 3) {
      const int c = fc + k0 + k;
      const S xc = fold4<S>(red, nout, (k > 0 ? k * nx + nU : 0) + lane);
      if (c < nl) put_tagged<S>(xt + ((size_t)c * nx + lane) * kTW<S>, xc, tag);
      zout[1 + (long long)c * nx + lane] = xc;
    }
  }
  __syncthreads();  // red and the matrices are reused by the next item
}

// ---------------------------------------------------------------- path piece
// Nodes node[0] .. node[m] (parent to child): x of node[0] from its forward
// item (x0 at the root), d of node[0] .. node[m - 1] from the backward items;
// then u = K x + d and x^c = Abar^c x + B^c d stage by stage, on wavefront 0.
// Nodes from node[own] on are this piece's to write. Wavefronts 0 and 3 copy
// the Abar, 1 the B, 2 K. The heads (B d, d) come from wavefront 1 for the top
// link, whose d is the last to arrive, and from 2 and 3 for the others.
template <typename S, int R, int SL>
__device__ __forceinline__ void walk_path(unsigned* lds, int rv) {
  const Args<S> A = here_args<S>();
  const int t = here_v(threadIdx.x), w = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  const int nx = here_s(A->P.nx), nu = here_s(A->P.nu), nl = A->P.nl, nout = nx + nu;
  const WalkLds L(nx, nu, A->nc, (int)(sizeof(S) / 4));
  constexpr int es = sizeof(S) / 4;
  const int m = rec_int(rv, 1), own = rec_int(rv, 2), top = rec_int(rv, 4);
  const S* M = reinterpret_cast<const S*>(lds);
  const int LW = L.path_link(), cK = L.sA + L.sB, cH = cK + (L.oQ - L.oK);
  {
    const S* mat = w == 1 ? A->P.BC : w == 2 ? A->P.KC : A->P.AbC;
    const int len = nx * (w == 1 || w == 2 ? nu : nx), off = w == 1 ? L.sA : w == 2 ? cK : 0;
    for (int l = w == 2 ? own : w == 3 ? 1 : 0; l < m; l += w == 1 || w == 2 ? 1 : 2)
      copy_in(mat + (size_t)rec_int(rv, w == 2 ? 4 + l : 5 + l) * len, lds, l * LW + off, len * es, lane);
  }
  wait_vm();
  __syncthreads();
  S x = 0;
  if (w == 0) {
    if (top != 0) {
      x = wait_lane<S>(A->xt + (size_t)top * nx * kTW<S>, nx, lane, A->tag, A->err, A->spin);
    } else if (lane < nx) {
      x = (S)A->x0[lane];
      if (own == 0) A->zout[1 + lane] = x;
    }
  } else {
    const LaneOut<1> X(nx, 0, lane);
    for (int l = w == 1 ? 0 : w - 1; l < (w == 1 ? 1 : m); l += 2) {
      const int f = rec_int(rv, 4 + l);
      const S d = wait_lane<S>(A->dt + (size_t)f * nu * kTW<S>, nu, lane, A->tag, A->err, A->spin);
      S a[1][2] = {};
      sum_rows<S, R, 1>(M, (l * LW + L.sA) / es, 0, X, nu, d, a);
      S* const h = reinterpret_cast<S*>(lds + l * LW + cH);
      if (lane < nx) h[lane] = a[0][0] + a[0][1];
      if (lane < nu) h[nx + lane] = d;
    }
  }
  __syncthreads();
  if (w == 0) {
    const LaneOut<SL> O(nx, nu, lane);
    S* const zout = A->zout;
    unsigned long long* const xt = A->xt;
    const unsigned tag = A->tag;
    const long long zU = A->P.zU;
    run_links<S, R, SL>(
        M, O, nx, nout, cK / es, lane, 0, m, x, [&](int l) { return l * LW / es; },
        [&](int l) { return (l * LW + cH) / es; },
        [&](int l, const S(&v)[SL]) {
          const int f = rec_int(rv, 4 + l), c = rec_int(rv, 5 + l);
          if (lane < nx && l + 1 >= own) {
            zout[1 + (long long)c * nx + lane] = v[0];
            if (l + 1 == m && c < nl) put_tagged<S>(xt + ((size_t)c * nx + lane) * kTW<S>, v[0], tag);
          }
          if (l >= own)
#pragma unroll
            for (int s = 0; s < SL; ++s) {
              const int o = lane + 64 * s;
              if (o >= nx && o < nout) zout[zU + (long long)f * nu + (o - nx)] = v[s];
            }
        });
  }
  __syncthreads();  // LDS reuse by the next item
}

// W: wavefronts per SIMD the register allocation targets.
template <typename S, int R, int SL, int W>
__global__ void __launch_bounds__(kFW) __attribute__((amdgpu_waves_per_eu(W, W))) k_T_walk(WalkArgs<S> A) {
  extern __shared__ __align__(16) unsigned walk_lds[];
  // items run in increasing order in every workgroup: its backward items,
  // then its forward items (two loops, so that the two kinds of item do not
  // hold registers at the same time); lane k holds entry k of an item's record
  const int lane = threadIdx.x & 63, e = lane < A.rs ? lane : A.rs - 1;
  int it = blockIdx.x;
  for (; it < A.nbwd; it += gridDim.x) walk_bwd<S, R, SL>(walk_lds, A.items[(size_t)it * A.rs + e]);
  for (; it < A.nitems; it += gridDim.x) {
    const int rv = A.items[(size_t)it * A.rs + e];
    if (rec_int(rv, 1) > 0)
      walk_path<S, R, SL>(walk_lds, rv);
    else
      walk_fwd<S, R, SL>(walk_lds, rv);
  }
}

// Wavefronts per SIMD of a build: what the held weights leave of the registers.
template <typename S, int R, int SL>
constexpr int kWaves = sizeof(S) / 4 * R * SL > 31 ? 2 : sizeof(S) / 4 * R * SL > 15 ? 3 : 4;

template <typename S, int R, int SL>
const void* walk_pick(int* waves) {
  if (waves) *waves = kWaves<S, R, SL>;
  return reinterpret_cast<const void*>(&k_T_walk<S, R, SL, kWaves<S, R, SL>>);
}

}  // namespace

// The build for the dimensions (rows per wavefront: a quarter of the larger,
// over the sizes built) and the wavefronts per SIMD it is compiled for. A size
// costs about what the largest of its build costs, since the rows past the end
// are multiplied too; six builds keep that within a fifth up to n_x 52, and the
// dataflow form is slower at every size (sweeps of 223 nodes in FP64, us, walk /
// dataflow: n_x 8 19.7 / 41, 9 21.7 / 42, 12 21.3 / 43, 13 24.4 / 44, 20 23.5 /
// 45, 21 28.4 / 46, 32 30 / 47, 33 35.5 / 50, 44 36 to 42 / 49 to 55, 52 41 / 52 to
// 57, 53 46 to 50 / 53 to 58, 64 43 / 54 to 60).
template <typename S>
const void* walk_kernel(int nx, int nu, int* waves) {
  const int n = std::max(nx, nu);
  if (n <= 8) return walk_pick<S, 2, 1>(waves);
  if (n <= 12) return walk_pick<S, 3, 1>(waves);
  if (n <= 20) return walk_pick<S, 5, 1>(waves);
  if (n <= 32) return walk_pick<S, 8, 1>(waves);
  if (n <= 52) return nx + nu <= 64 ? walk_pick<S, 13, 1>(waves) : walk_pick<S, 13, 2>(waves);
  return nx + nu <= 64 ? walk_pick<S, 16, 1>(waves) : walk_pick<S, 16, 2>(waves);
}
template const void* walk_kernel<double>(int, int, int*);
template const void* walk_kernel<float>(int, int, int*);

// LDS bytes of the launch with nc children per chunk, chains of chain links
// and path pieces of path links.
int walk_lds_bytes(int nx, int nu, int nc, int elem, int chain, int path) {
  const WalkLds L(nx, nu, nc, elem / 4);
  return 4 * std::max(L.words + (chain - 1) * L.chain_link(), path * L.path_link());
}

template <typename S>
hipError_t launch_sweeps_walk(const Problem& P, const DevProb<S>& D, S* zout, const double* x0, const S* xbar,
                              const S* ubar, const S* q, hipStream_t st) {
  const FlowState& F = P.walk;
  if (!F.qt || F.grid <= 0) return hipErrorInvalidValue;
  WalkArgs<S> A;
  A.P = D;
  A.zout = zout;
  A.x0 = x0;
  A.xbar = xbar;
  A.ubar = ubar;
  A.seeds = q;
  A.qt = F.qt;
  A.dt = F.dt;
  A.xt = F.xt;
  A.pt = F.pt;
  A.items = F.items;
  A.pbase = F.pbase;
  A.err = P.flow_err;
  A.spin = F.spin;
  if (++P.flow_epoch == 0u) P.flow_epoch = 1u;  // tag 0 is the cleared state
  A.tag = P.flow_epoch;
  A.nc = F.nc;
  A.nbwd = F.nbwd;
  A.nitems = F.nitems;
  A.rs = F.rs;
  void* args[] = {&A};
  const void* k = walk_kernel<S>(P.nx, P.nu, nullptr);
  const dim3 grid(std::min(F.grid, F.nitems));
  return F.coop ? hipLaunchCooperativeKernel(k, grid, dim3(kFW), args, (unsigned)F.lds, st)
                : hipLaunchKernel(k, grid, dim3(kFW), args, (size_t)F.lds, st);
}
template hipError_t launch_sweeps_walk<double>(const Problem&, const DevProb<double>&, double*, const double*,
                                               const double*, const double*, const double*, hipStream_t);
template hipError_t launch_sweeps_walk<float>(const Problem&, const DevProb<float>&, float*, const double*,
                                              const float*, const float*, const float*, hipStream_t);

}  // namespace spk
