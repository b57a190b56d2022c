// Fine-lattice kernels: layout transforms, clover term, the twisted-mass
// Wilson-clover operator D(mu) = D_W + i mu Gamma5 (paper Sec. 1), the SAP
// smoother with odd-even block MR (Sec. 1 smoother, Sec. 3 odd-even in the
// smoother), Gamma5-compatible restriction / prolongation and block
// orthonormalisation (Sec. 1 aggregation), and the Galerkin assembly of the
// first coarse operator D_c = P^dag D_W P (Sec. 1, Eq. 1 context).
//
// Operator conventions (the paper fixes gamma5 = diag(-1,-1,1,1) and TZYX
// order only):
//   (D psi)(x) = T(x) psi(x) - 1/2 sum_mu [(1-g_mu) U_mu(x) psi(x+mu)
//                                        + (1+g_mu) U_mu(x-mu)^dag psi(x-mu)]
//   T(x) = (m0+4) + A(x) + i tw gamma5,   A = (i c_sw/4) sum sigma_{mu nu} F_{mu nu}
// Chiral gamma basis: g_k = [[0,-i s_k],[i s_k,0]] (k = X,Y,Z), g_T = [[0,-1],[-1,0]].
// With g_mu = [[0,B],[B^dag,0]] the projector (1 -+ g_mu) has rank 2: only the
// half spinor h = psi_up -+ B psi_dn is transported by U, the lower half is
// rebuilt from it.  Per direction and sign the reconstruction is a pair of
// phases in {1, i, -1, -i} and a spin permutation (tables below).
#include "finedev.hpp"


namespace ddamg {



// ---------------------------------------------------------------------------
// workgroup reduction helpers (deterministic: fixed shuffle and wave order)

// ---------------------------------------------------------------------------
// SAP: one colour sweep.  One workgroup per block of the colour, one thread per
// slot (even slots first).  r = b - D x on the block, then n_mr MR steps
// on the block-local even-site Schur complement S = T_ee - D_eo T_oo^{-1} D_oe
// (hops leaving the block dropped), odd reconstruction, x += e.

// In-block neighbours of a slot, packed: for direction mu the forward and the
// backward neighbour's index within the other parity's half of the block
// (bytes 2(mu&1) and 2(mu&1)+1 of word mu>>1), or `half` where the hop
// leaves the block.  Computed once per thread; the block solve reads its
// neighbours from LDS halves whose index `half` holds a zero spinor, so a
// dropped hop costs neither an index computation nor a mask.
struct BlockNbr {
  unsigned w[2];
};
__device__ __forceinline__ BlockNbr block_nbrs(const Geom& g, const SiteNbr& me) {
  BlockNbr nb{{0u, 0u}};
#pragma unroll
  for (int mu = 0; mu < 4; ++mu) {
    int l[4] = {me.l[0], me.l[1], me.l[2], me.l[3]};
    const int l0 = l[mu];
    int f = g.half, b = g.half;
    if (l0 + 1 < g.b[mu]) {
      l[mu] = l0 + 1;
      const int sn = local_slot(g, l);
      f = sn >= g.half ? sn - g.half : sn;
    }
    if (l0 > 0) {
      l[mu] = l0 - 1;
      const int sn = local_slot(g, l);
      b = sn >= g.half ? sn - g.half : sn;
    }
    nb.w[mu >> 1] |= (unsigned)(f | (b << 8)) << (16 * (mu & 1));
  }
  return nb;
}

// The block solve's fields in LDS: entry idx of component pair p at p * hs + idx,
// so that a site is six 16-byte (FP32) accesses of consecutive entries.
template <class R>
struct alignas(4 * sizeof(R)) cxpair {
  cx<R> a, b;
};
template <class R, bool NEG = false, int NP = 6>
__device__ __forceinline__ void pair_get(const cxpair<R>* f, int hs, int idx, cx<R>* v) {
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const cxpair<R> q = f[p * hs + idx];
    v[2 * p] = NEG ? -q.a : q.a;
    v[2 * p + 1] = NEG ? -q.b : q.b;
  }
}
template <class R, int NP = 6>
__device__ __forceinline__ void pair_put(cxpair<R>* f, int hs, int idx, const cx<R>* v) {
#pragma unroll
  for (int p = 0; p < NP; ++p) f[p * hs + idx] = cxpair<R>{v[2 * p], v[2 * p + 1]};
}

// the links of direction MU's two in-block hops at a slot; a dropped backward hop
// reads a link of the block, multiplied by the zero spinor
template <int MU, class S>
__device__ __forceinline__ void hop_block_load(const typename store_traits<S>::elem* U, const Geom& g, int B,
                                               long site_s, BlockNbr nb, int noff, RawLink<S>& cf, RawLink<S>& cb) {
  const int sb = (nb.w[MU >> 1] >> (16 * (MU & 1) + 8)) & 255;
  load_raw<S>(U, site_s, MU, cf);
  load_raw<S>(U, link_site<S>(g, B, min(sb, g.half - 1) + noff), MU, cb);
}
template <int MU, class R, class S, bool SUB>
__device__ __forceinline__ void hop_block_dir(const RawLink<S>& cf, const RawLink<S>& cb, const cxpair<R>* lds,
                                              int hs, BlockNbr nb, cx<R> out[12]) {
  const unsigned wd = nb.w[MU >> 1] >> (16 * (MU & 1));
  const int sf = wd & 255, sb = (wd >> 8) & 255;
  cx<R> psi[12], u[9];
  unpack_link<MU, R, S>(cf, u);
  pair_get<R, SUB>(lds, hs, sf, psi);
  hop_accum_t<0, MU>(psi, u, out);
  unpack_link<MU, R, S>(cb, u);
  pair_get<R, SUB>(lds, hs, sb, psi);
  hop_accum_t<1, MU>(psi, u, out);
}
// out += (or -= with SUB) the in-block hops of slot s, the neighbours' spinors
// read from lds (the other parity's half of the block; entry `half` of every
// pair is zero).  noff: slot offset of the neighbours' parity (their links are
// read for the backward hops).  `last`: loads to issue before the last
// direction multiplies.
template <class R, class S, bool SUB = false, class F>
__device__ __forceinline__ void hop_block_lds(const typename store_traits<S>::elem* U, const Geom& g, int B, int s,
                                              BlockNbr nb, int noff, const cxpair<R>* lds, int hs, cx<R> out[12],
                                              F last) {
  // opaque per call: nothing derived from the neighbour words or the slot is
  // kept live across the MR steps
  __asm__ volatile("" : "+v"(nb.w[0]), "+v"(nb.w[1]), "+v"(s));
  const long site_s = link_site<S>(g, B, s);
  RawLink<S> cf, cb, nf, nn;
  hop_block_load<0, S>(U, g, B, site_s, nb, noff, cf, cb);
  // the links of the next direction are in flight while this one multiplies; the
  // scheduling barriers keep the later directions' loads from being hoisted
  hop_block_load<1, S>(U, g, B, site_s, nb, noff, nf, nn);
  __builtin_amdgcn_sched_barrier(0);
  hop_block_dir<0, R, S, SUB>(cf, cb, lds, hs, nb, out);
  __builtin_amdgcn_sched_barrier(0);
  hop_block_load<2, S>(U, g, B, site_s, nb, noff, cf, cb);
  __builtin_amdgcn_sched_barrier(0);
  hop_block_dir<1, R, S, SUB>(nf, nn, lds, hs, nb, out);
  __builtin_amdgcn_sched_barrier(0);
  hop_block_load<3, S>(U, g, B, site_s, nb, noff, nf, nn);
  __builtin_amdgcn_sched_barrier(0);
  hop_block_dir<2, R, S, SUB>(cf, cb, lds, hs, nb, out);
  __builtin_amdgcn_sched_barrier(0);
  last();
  __builtin_amdgcn_sched_barrier(0);
  hop_block_dir<3, R, S, SUB>(nf, nn, lds, hs, nb, out);
}
template <class R, class S, bool SUB = false>
__device__ __forceinline__ void hop_block_lds(const typename store_traits<S>::elem* U, const Geom& g, int B, int s,
                                              BlockNbr nb, int noff, const cxpair<R>* lds, int hs, cx<R> out[12]) {
  hop_block_lds<R, S, SUB>(U, g, B, s, nb, noff, lds, hs, out, [] {});
}

// w = T_oo^{-1} (in-block hops of the other parity's field in lds) at odd slot s.
// FP32: the rows of T_oo^{-1} are loaded three ahead of their products, the first
// during the last direction of the hops.
template <class R, class S>
__device__ __forceinline__ void hop_inv_block(const typename store_traits<S>::elem* U, const R* H, const R* Minv,
                                              const Geom& g, int B, int s, TwistR<R> tw, BlockNbr nb,
                                              const cxpair<R>* lds, int hs, cx<R> w[12]) {
  cx<R> u[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) u[c] = mk<R>(0, 0);
  if constexpr (sizeof(R) == 8) {
    hop_block_lds<R, S>(U, g, B, s, nb, 0, lds, hs, u);
    site_inv(H, Minv, g, B, s, tw, u, w);
  } else {
    const int io = s - g.half, tl = io % TILE;
    const long tt = (long)B * (g.half / TILE) + io / TILE;
    TinvRows a, b;
    hop_block_lds<R, S>(U, g, B, s, nb, 0, lds, hs, u, [&] { tinv_load(Minv, tt, tl, 0, a); });
    __builtin_amdgcn_sched_barrier(0);
    tinv_load(Minv, tt, tl, 1, b);
    __builtin_amdgcn_sched_barrier(0);
    tinv_mv(a, u, w);
    __builtin_amdgcn_sched_barrier(0);
    tinv_load(Minv, tt, tl, 2, a);
    __builtin_amdgcn_sched_barrier(0);
    tinv_mv(b, u, w + 3);
    __builtin_amdgcn_sched_barrier(0);
    tinv_load(Minv, tt, tl, 3, b);
    __builtin_amdgcn_sched_barrier(0);
    tinv_mv(a, u + 6, w + 6);
    tinv_mv(b, u + 6, w + 9);
  }
}

// SAP colour sweep.  One workgroup per block of the colour (and field), one
// thread per pair of slots: thread i owns even slot i and odd slot half + i,
// so both wavefronts of a block have work in the even-site and in the
// odd-site half of every MR step.
//   r = b - D x on the block;  t_o = T_oo^{-1} r_o,  x_o += t_o;
//   rho = r_e - D_eo t_o;  n_mr MR steps on S = T_ee - D_eo T_oo^{-1} D_oe
//   (block-local hops only) accumulate e_e;  x_e += e_e,
//   x_o -= T_oo^{-1} D_oe e_e  (together: x_o += T_oo^{-1} (r_o - D_oe e_e)).
// x of a block is read and written by its own workgroup only: the residual
// reads the other colour's blocks, which this sweep leaves unchanged.
// Bound by the vector units (at 48x24^3, six fields, 16-bit links, 4 MR steps
// they issue in about 85 % of the cycles of two wavefronts per SIMD; the links,
// clover and inverses of a block come from L2 after the first MR step), so the
// levers are fewer instructions and no idle issue slots: unrolled directions with
// compile-time spin projections, T_oo^{-1} as one product, 16-byte loads and LDS
// accesses, each direction's links and each three rows of T_oo^{-1} loaded while
// those before multiply.  1042 -> 769 us a sweep there, 105 -> 84 us
// with one field and FP32 links at 24x16x16x24.  All 256 registers are in use:
// with 168 (three wavefronts per SIMD) these take 1086 and 129 us.  Small grids, and
// one field with FP32 links on blocks that fill its wavefronts, take k_sap_two.
template <class R, class S>
__global__ void __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 ? 1 : 2, 8)))
k_sap(Geom g, int colour, const typename store_traits<S>::elem* __restrict__ U, const R* __restrict__ H,
      const R* __restrict__ Minv, TwistR<R> tw, const cx<R>* __restrict__ b, cx<R>* __restrict__ x, int n_mr, int K,
      long ld) {
  extern __shared__ char smem_raw[];
  // the residual stages x of the block parity-split (24 x half); the block
  // solve then keeps one field per parity as 6 pairs x hs (hs = half + 1: entry
  // half is the zero spinor of dropped hops)
  const int hs = g.half + 1;
  cx<R>* xs = reinterpret_cast<cx<R>*>(smem_raw);
  cxpair<R>* ev = reinterpret_cast<cxpair<R>*>(smem_raw);  // even slots
  cxpair<R>* od = ev + 6 * hs;                              // odd slots
  __shared__ double red[2][3][2];                    // per-wavefront sums, by MR step parity
  int B;
  {
    // K right-hand sides interleaved: consecutive workgroups (same XCD) take
    // the same lattice block for different fields, so its links, clover and
    // odd-site inverses are shared through L2
    const int w = xcd_remap(blockIdx.x, gridDim.x);
    const int pair = w / K, rr = w - pair * K;
    b += (long)rr * ld;
    x += (long)rr * ld;
    int B0 = 2 * pair;
    int bc[4];
    block_coords(g, B0, bc);
    int par = (bc[0] + bc[1] + bc[2] + bc[3]) & 1;
    B = B0 + ((par ^ colour) & 1);
  }
  const int i = threadIdx.x;
  const int se = i, so = g.half + i;
  const int lane = i & 63, wv = i >> 6, nw = (g.half + 63) >> 6;
  SiteNbr me_e, me_o;
  me_of(g, B, se, me_e);
  me_of(g, B, so, me_o);
  cx<R> rho[12], ee[12], tmp[12];
  {
    // r = b - D x with x of this block staged in ev/od
    cx<R> psi[12], ro[12];
    load_spinor(x, g, B, se, psi);
#pragma unroll
    for (int c = 0; c < 12; ++c) *lds_site(xs, g, se, c) = psi[c];
    site_term(H, g, B, se, tw, psi, rho);
    __asm__ volatile("" ::: "memory");
    load_spinor(x, g, B, so, psi);
#pragma unroll
    for (int c = 0; c < 12; ++c) *lds_site(xs, g, so, c) = psi[c];
    site_term(H, g, B, so, tw, psi, ro);
    __syncthreads();
    hop_staged<R, S>(U, x, xs, g, B, se, me_e, rho);
    __asm__ volatile("" ::: "memory");
    hop_staged<R, S>(U, x, xs, g, B, so, me_o, ro);
    load_spinor(b, g, B, se, psi);
#pragma unroll
    for (int c = 0; c < 12; ++c) rho[c] = psi[c] - rho[c];
    load_spinor(b, g, B, so, psi);
#pragma unroll
    for (int c = 0; c < 12; ++c) ro[c] = psi[c] - ro[c];
    __syncthreads();
    __asm__ volatile("" ::: "memory");
    site_inv(H, Minv, g, B, so, tw, ro, tmp);
    load_spinor(x, g, B, so, psi);
    pair_put(od, hs, i, tmp);
#pragma unroll
    for (int c = 0; c < 12; ++c) psi[c] += tmp[c];
    store_spinor(x, g, B, so, psi);
    for (int e = i; e < 12; e += g.half) ev[e * hs + g.half] = cxpair<R>{mk<R>(0, 0), mk<R>(0, 0)};  // od follows ev
  }
  const BlockNbr nb_e = block_nbrs(g, me_e), nb_o = block_nbrs(g, me_o);
  __syncthreads();
  hop_block_lds<R, S, true>(U, g, B, se, nb_e, g.half, od, hs, rho);  // rho = r_e - D_eo t_o
#pragma unroll
  for (int c = 0; c < 12; ++c) ee[c] = mk<R>(0, 0);
  const int nact = min(64, g.half - wv * 64);
  pair_put(ev, hs, i, rho);
  for (int k = 0; k < n_mr; ++k) {
    // the block operator is re-read in every step: keeping the loop-invariant
    // links, clover and inverses in registers would exceed the register file;
    // rho lives in LDS, where the neighbours read it anyway
    __asm__ volatile("" ::: "memory");
    __syncthreads();
    // w = T_oo^{-1} D_oe rho
    hop_inv_block<R, S>(U, H, Minv, g, B, so, tw, nb_o, ev, hs, tmp);
    pair_put(od, hs, i, tmp);
    __syncthreads();
    __asm__ volatile("" ::: "memory");
    // q = T_ee rho - D_eo w
    pair_get(ev, hs, i, rho);
    site_term(H, g, B, se, tw, rho, tmp);
    __asm__ volatile("" ::: "memory");
    hop_block_lds<R, S, true>(U, g, B, se, nb_e, g.half, od, hs, tmp);
    double qr_re = 0, qr_im = 0, qq = 0;
    __asm__ volatile("" ::: "memory");
    pair_get(ev, hs, i, rho);
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      qr_re += (double)tmp[c].re * rho[c].re + (double)tmp[c].im * rho[c].im;
      qr_im += (double)tmp[c].re * rho[c].im - (double)tmp[c].im * rho[c].re;
      qq += (double)tmp[c].re * tmp[c].re + (double)tmp[c].im * tmp[c].im;
    }
    qr_re = wave_sum_n(qr_re, nact);
    qr_im = wave_sum_n(qr_im, nact);
    qq = wave_sum_n(qq, nact);
    if (lane == 0) {
      red[k & 1][0][wv] = qr_re;
      red[k & 1][1][wv] = qr_im;
      red[k & 1][2][wv] = qq;
    }
    __syncthreads();
    double sr = 0, si = 0, sq = 0;
    for (int v = 0; v < nw; ++v) {
      sr += red[k & 1][0][v];
      si += red[k & 1][1][v];
      sq += red[k & 1][2][v];
    }
    cx<R> alpha = mk<R>(0, 0);
    if (sq > 0) alpha = mk<R>((R)(sr / sq), (R)(si / sq));
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      ee[c] += alpha * rho[c];
      rho[c] -= alpha * tmp[c];
    }
    pair_put(ev, hs, i, rho);
  }
  pair_put(ev, hs, i, ee);
  __syncthreads();
  {  // x_o -= T_oo^{-1} D_oe e_e
    cx<R> u[12];
    hop_inv_block<R, S>(U, H, Minv, g, B, so, tw, nb_o, ev, hs, tmp);
    load_spinor(x, g, B, so, u);
#pragma unroll
    for (int c = 0; c < 12; ++c) u[c] -= tmp[c];
    store_spinor(x, g, B, so, u);
  }
  load_spinor(x, g, B, se, tmp);
#pragma unroll
  for (int c = 0; c < 12; ++c) tmp[c] += ee[c];
  store_spinor(x, g, B, se, tmp);
}

// The two threads of a site pair: thread `part` takes directions 2 part and
// 2 part + 1 of every hop sum and chirality `part` of everything diagonal in
// it.  A hop sum's halves meet through LDS: each thread hands over its partial
// sums of the other chirality (ex: [chirality][3 pairs][stride]) and keeps its
// own; ends with the sum, and contains one barrier.
__device__ __forceinline__ void exchange_halves(cxpair<float>* ex, int stride, int i, int part, bool live, const cx<float> v[12],
                                                cx<float> own[6]) {
  cx<float> give[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    own[c] = part ? v[6 + c] : v[c];
    give[c] = part ? v[c] : v[6 + c];
  }
  if (live) pair_put<float, 3>(ex + (part ? 0 : 3) * stride, stride, i, give);
  __syncthreads();
  pair_get<float, false, 3>(ex + (part ? 3 : 0) * stride, stride, i, give);
#pragma unroll
  for (int c = 0; c < 6; ++c) own[c] += give[c];
}

// a thread's links of a slot's in-block hops: forward and backward, its two directions
template <class S>
struct PartLinks {
  RawLink<S> f[2], b[2];
};
template <class S>
__device__ __forceinline__ void part_links(const typename store_traits<S>::elem* U, const Geom& g, int B, int s,
                                           BlockNbr nb, int noff, int part, PartLinks<S>& l) {
  const long site_s = link_site<S>(g, B, s);
  const unsigned wd = part ? nb.w[1] : nb.w[0];
#pragma unroll
  for (int d = 0; d < 2; ++d) {
    const int sb = (wd >> (16 * d + 8)) & 255;
    load_raw<S>(U, site_s, 2 * part + d, l.f[d]);
    load_raw<S>(U, link_site<S>(g, B, min(sb, g.half - 1) + noff), 2 * part + d, l.b[d]);
  }
}
// FP16: a copy whose conversion stays where it is used; hoisted out of the MR steps
// the converted links spill (BF16 links do not, and take 36.9 us so, 38.5 this way)
template <class S>
__device__ __forceinline__ RawLink<S> use_link(RawLink<S> r) {
  if constexpr (std::is_same<S, f16>::value) {
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
      for (int w = 0; w < 4; ++w) __asm__ volatile("" : "+v"(r.c[c].w[w]));
  }
  return r;
}
// own += (or -= with SUB) this thread's chirality of the in-block hops of its slot,
// the other parity's field in lds
template <class S, bool SUB>
__device__ __forceinline__ void hop_two(const PartLinks<S>& l, const Geom& g, BlockNbr nb, const cxpair<float>* lds,
                                        int hs, cxpair<float>* ex, int i, int part, bool live, cx<float> own[6]) {
  cx<float> h[12], sum[6];
#pragma unroll
  for (int c = 0; c < 12; ++c) h[c] = mk<float>(0, 0);
  if (part == 0) {
    hop_block_dir<0, float, S, SUB>(use_link<S>(l.f[0]), use_link<S>(l.b[0]), lds, hs, nb, h);
    hop_block_dir<1, float, S, SUB>(use_link<S>(l.f[1]), use_link<S>(l.b[1]), lds, hs, nb, h);
  } else {
    hop_block_dir<2, float, S, SUB>(use_link<S>(l.f[0]), use_link<S>(l.b[0]), lds, hs, nb, h);
    hop_block_dir<3, float, S, SUB>(use_link<S>(l.f[1]), use_link<S>(l.b[1]), lds, hs, nb, h);
  }
  exchange_halves(ex, g.half, i, part, live, h, sum);
#pragma unroll
  for (int c = 0; c < 6; ++c) own[c] += sum[c];
}
// chirality block `part` of T psi and of T^{-1} psi
__device__ __forceinline__ void term_two(const float h[36], int part, float tw, const cx<float> psi[6],
                                         cx<float> out[6]) {
  const float t = part ? tw : -tw;
  herm_mv(h, 1, psi, out);
#pragma unroll
  for (int c = 0; c < 6; ++c) out[c] += t * times_i(psi[c]);
}
__device__ __forceinline__ void inv_two(const TinvRows r[2], const cx<float> psi[6], cx<float> out[6]) {
  tinv_mv(r[0], psi, out);
  tinv_mv(r[1], psi, out + 3);
}

// The sweep for grids that leave most of the chip idle, and for one field with FP32
// links on large blocks: two threads for a pair of slots, in wavefronts of their own, and a
// wavefront alone on its SIMD.  Bound by the chain of an MR step (two hop sums, two
// exchanges, the dots), so that is what is halved, and the operator entries of a
// thread (200 to 250 registers) are loaded once and stay in the register file of
// 512 through the MR steps.  Sizes measured: sap_two.
template <class S>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2)))
k_sap_two(Geom g, int colour, const typename store_traits<S>::elem* __restrict__ U, const float* __restrict__ H,
          const float* __restrict__ Tinv, TwistR<float> tw, const cx<float>* __restrict__ b, cx<float>* __restrict__ x,
          int n_mr, int K, long ld) {
  extern __shared__ char smem_raw[];
  // the residual stages x of the block parity-split (24 x half); the block
  // solve then keeps one field per parity as 6 pairs x hs (hs = half + 1: entry
  // half is the zero spinor of dropped hops), and the halves of a hop sum pass
  // through ex
  const int hs = g.half + 1;
  cx<float>* xs = reinterpret_cast<cx<float>*>(smem_raw);
  cxpair<float>* ev = reinterpret_cast<cxpair<float>*>(smem_raw);  // even slots
  cxpair<float>* od = ev + 6 * hs;                                  // odd slots
  cxpair<float>* ex = od + 6 * hs;                                  // 6 x half
  __shared__ double red[2][3][4];                                   // per-wavefront sums, by MR step parity
  int B;
  {
    // K right-hand sides interleaved: consecutive workgroups (same XCD) take
    // the same lattice block for different fields, so its links, clover and
    // odd-site inverses are shared through L2
    const int w = xcd_remap(blockIdx.x, gridDim.x);
    const int pair = w / K, rr = w - pair * K;
    b += (long)rr * ld;
    x += (long)rr * ld;
    int B0 = 2 * pair;
    int bc[4];
    block_coords(g, B0, bc);
    int par = (bc[0] + bc[1] + bc[2] + bc[3]) & 1;
    B = B0 + ((par ^ colour) & 1);
  }
  const int nt = blockDim.x >> 1;  // threads of one part: half rounded up to wavefronts
  const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >= nt ? 1 : 0);
  const int i0 = threadIdx.x - part * nt;
  const bool live = i0 < g.half;
  // threads past the block's slots follow the last one and store nothing
  const int i = live ? i0 : g.half - 1;
  const int se = i, so = g.half + i;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const long oe = fidx(g, B, se, 12) + (long)(6 * part) * TILE, oo = fidx(g, B, so, 12) + (long)(6 * part) * TILE;
  SiteNbr me_e, me_o;
  me_of(g, B, se, me_e);
  me_of(g, B, so, me_o);
  cx<float> rho[6], ee[6], tmp[6];
  // the block operator of the thread's two slots stays in registers
  const BlockNbr nb_e = block_nbrs(g, me_e), nb_o = block_nbrs(g, me_o);
  float he[36];
  TinvRows ti[2];
  PartLinks<S> le, lo;
  herm_load(H, (long)B * (g.bs / TILE) + se / TILE, se % TILE, part, he);
  {
    // r = b - D x with x of this block staged in LDS
    cx<float> ro[6], xe[6], xo[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      xe[c] = x[oe + (long)c * TILE];
      xo[c] = x[oo + (long)c * TILE];
    }
    if (live) {
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        *lds_site(xs, g, se, 6 * part + c) = xe[c];
        *lds_site(xs, g, so, 6 * part + c) = xo[c];
      }
    }
    term_two(he, part, tw.e, xe, rho);
    {
      float ho[36];
      herm_load(H, (long)B * (g.bs / TILE) + so / TILE, so % TILE, part, ho);
      term_two(ho, part, tw.o, xo, ro);
    }
    __syncthreads();
    cx<float> h[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) h[c] = mk<float>(0, 0);
    hop_staged<float, S>(U, x, xs, g, B, se, me_e, h, 2 * part, 2 * part + 2);
    exchange_halves(ex, g.half, i, part, live, h, tmp);
#pragma unroll
    for (int c = 0; c < 6; ++c) rho[c] = b[oe + (long)c * TILE] - (rho[c] + tmp[c]);
#pragma unroll
    for (int c = 0; c < 12; ++c) h[c] = mk<float>(0, 0);
    hop_staged<float, S>(U, x, xs, g, B, so, me_o, h, 2 * part, 2 * part + 2);
    __syncthreads();  // the first exchange has been read
    exchange_halves(ex, g.half, i, part, live, h, tmp);
#pragma unroll
    for (int c = 0; c < 6; ++c) ro[c] = b[oo + (long)c * TILE] - (ro[c] + tmp[c]);
    // (every thread has passed the exchange's barrier: xs is free)
#pragma unroll
    for (int q = 0; q < 2; ++q)
      tinv_load(Tinv, (long)B * (g.half / TILE) + i / TILE, i % TILE, 2 * part + q, ti[q]);
    part_links<S>(U, g, B, se, nb_e, g.half, part, le);
    part_links<S>(U, g, B, so, nb_o, 0, part, lo);
    inv_two(ti, ro, tmp);
    if (live) {
      pair_put<float, 3>(od + 3 * part * hs, hs, i, tmp);
#pragma unroll
      for (int c = 0; c < 6; ++c) x[oo + (long)c * TILE] = xo[c] + tmp[c];
    }
    // od follows ev: 12 rows whose entry `half` is zero
    if (threadIdx.x < 12) ev[threadIdx.x * hs + g.half] = cxpair<float>{mk<float>(0, 0), mk<float>(0, 0)};
  }
  __syncthreads();
  // rho = r_e - D_eo t_o
  hop_two<S, true>(le, g, nb_e, od, hs, ex, i, part, live, rho);
#pragma unroll
  for (int c = 0; c < 6; ++c) ee[c] = mk<float>(0, 0);
  cxpair<float>* evp = ev + 3 * part * hs;
  cxpair<float>* odp = od + 3 * part * hs;
  if (live) pair_put<float, 3>(evp, hs, i, rho);
  for (int k = 0; k < n_mr; ++k) {
    __syncthreads();
    {  // w = T_oo^{-1} D_oe rho
      cx<float> u[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) u[c] = mk<float>(0, 0);
      hop_two<S, false>(lo, g, nb_o, ev, hs, ex, i, part, live, u);
      inv_two(ti, u, tmp);
      if (live) pair_put<float, 3>(odp, hs, i, tmp);
    }
    __syncthreads();
    // q = T_ee rho - D_eo w
    term_two(he, part, tw.e, rho, tmp);
    hop_two<S, true>(le, g, nb_e, od, hs, ex, i, part, live, tmp);
    double qr_re = 0, qr_im = 0, qq = 0;
    if (live) {
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        qr_re += (double)tmp[c].re * rho[c].re + (double)tmp[c].im * rho[c].im;
        qr_im += (double)tmp[c].re * rho[c].im - (double)tmp[c].im * rho[c].re;
        qq += (double)tmp[c].re * tmp[c].re + (double)tmp[c].im * tmp[c].im;
      }
    }
    qr_re = wave_sum_n(qr_re, 64);
    qr_im = wave_sum_n(qr_im, 64);
    qq = wave_sum_n(qq, 64);
    if (lane == 0) {
      red[k & 1][0][wv] = qr_re;
      red[k & 1][1][wv] = qr_im;
      red[k & 1][2][wv] = qq;
    }
    __syncthreads();
    double sr = 0, si = 0, sq = 0;
    for (int v = 0; v < nw; ++v) {
      sr += red[k & 1][0][v];
      si += red[k & 1][1][v];
      sq += red[k & 1][2][v];
    }
    cx<float> alpha = mk<float>(0, 0);
    if (sq > 0) alpha = mk<float>((float)(sr / sq), (float)(si / sq));
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      ee[c] += alpha * rho[c];
      rho[c] -= alpha * tmp[c];
    }
    if (live) pair_put<float, 3>(evp, hs, i, rho);
  }
  if (live) pair_put<float, 3>(evp, hs, i, ee);
  __syncthreads();
  {  // x_o -= T_oo^{-1} D_oe e_e
    cx<float> u[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) u[c] = mk<float>(0, 0);
    hop_two<S, false>(lo, g, nb_o, ev, hs, ex, i, part, live, u);
    inv_two(ti, u, tmp);
  }
  if (!live) return;
#pragma unroll
  for (int c = 0; c < 6; ++c) x[oo + (long)c * TILE] = x[oo + (long)c * TILE] - tmp[c];
#pragma unroll
  for (int c = 0; c < 6; ++c) x[oe + (long)c * TILE] = x[oe + (long)c * TILE] + ee[c];
}

// Whether a sweep of nwg workgroups takes k_sap_two (us a sweep, k_sap and it).
// While every SIMD has at most one wavefront of it (two or four a workgroup), the
// shorter chain wins for every block: 8x8x8x16 54 and 37 with 16-bit links, 57 and
// 38 with FP32, 432 workgroups of 8 pairs 97 and 39, 512 of 32 pairs 61 and 40, 256 of
// 128 pairs 58 and 40; past that its second round costs more (288 of 128 pairs 74
// and 82, six fields on 16^4 73 and 117).  Blocks of 8 pairs: k_sap's workgroups
// are one short wavefront, and up to about 1000 of them the dispatcher puts some in
// twos on a SIMD while others idle (648: 41 % of the wavefront cycles wait for the
// issue slot), so that two rounds of this kernel still win: 864 146 and 75, 1152 90
// and 113; with FP16 links three nearly do, 1152 145 and 107, 1296 126 and 107, 1536
// 108 and 109.
// One field with FP32 links of large blocks is bound by reading the operator again
// in every step, so there it also wins once the rounds are full, if most lanes of
// its wavefronts have a pair: 64 pairs 864 workgroups 102 and 83, 5120 627 and 463;
// 104 pairs 1200 264 and 227; 128 pairs 432 100 and 88, 3200 789 and 623; 56 and
// 112 pairs within these.  At three quarters (48 and 96 pairs) only from 6000
// wavefronts on: 1728 of 48 pairs 161 and 166, 3456 340 and 301.  Emptier
// wavefronts multiply by nothing: 8 pairs 16464 workgroups 813 and 1263, 24 pairs
// 5184 306 and 438, 32 pairs 4608 315 and 375, 72 pairs 2592 378 and 477, 88 pairs
// 3136 554 and 579.
template <class S>
static inline bool sap_two(const Geom& g, int nwg, int K) {
  const int slots = (g.half + 63) / 64 * 64;  // lanes of a part; g.half of them have a pair
  const long waves = (long)nwg * (slots / 32);
  if (waves <= (g.half > 8 ? 1024 : std::is_same<S, f16>::value ? 2816 : 2048)) return true;
  if (sizeof(S) != 4 || K != 1) return false;
  return 4 * g.half > 3 * slots ? waves >= 1536 : 4 * g.half == 3 * slots && waves >= 6144;
}
template <class R, class S>
void launch_sap(const Geom& g, int colour, const void* U, const R* H, const R* Tinv, Twist tw, const cx<R>* b,
                cx<R>* x, int n_mr, hipStream_t st) {
  launch_sap_multi<R, S>(g, colour, U, H, Tinv, tw, b, x, n_mr, 1, 0, st);
}
template <class R, class S>
void launch_sap_multi(const Geom& g, int colour, const void* U, const R* H, const R* Tinv, Twist tw, const cx<R>* b,
                      cx<R>* x, int n_mr, int K, long ld, hipStream_t st) {
  if constexpr (sizeof(R) == 4) {
    if (sap_two<S>(g, (g.nblocks / 2) * K, K)) {
      // ev and od (which the staged x, 24 half entries, fits in) and ex
      const size_t sm = (12 * (size_t)(g.half + 1) + 6 * (size_t)g.half) * sizeof(cxpair<float>);
      hipLaunchKernelGGL(k_sap_two<S>, dim3((g.nblocks / 2) * K), dim3(2 * ((g.half + 63) / 64 * 64)), sm, st, g, colour,
                         (const typename store_traits<S>::elem*)U, H, Tinv, TwistR<R>(tw), b, x, n_mr, K, ld);
      return;
    }
  }
  size_t sm = 2 * 12 * (size_t)(g.half + 1) * sizeof(cx<R>);
  hipLaunchKernelGGL((k_sap<R, S>), dim3((g.nblocks / 2) * K), dim3(g.half), sm, st, g, colour,
                     (const typename store_traits<S>::elem*)U, H, Tinv, TwistR<R>(tw), b, x, n_mr, K, ld);
}
template void launch_sap_multi<double, double>(const Geom&, int, const void*, const double*, const double*, Twist,
                                               const cx<double>*, cx<double>*, int, int, long, hipStream_t);
template void launch_sap_multi<float, float>(const Geom&, int, const void*, const float*, const float*, Twist,
                                             const cx<float>*, cx<float>*, int, int, long, hipStream_t);
template void launch_sap_multi<float, f16>(const Geom&, int, const void*, const float*, const float*, Twist,
                                           const cx<float>*, cx<float>*, int, int, long, hipStream_t);
template void launch_sap_multi<float, bf16>(const Geom&, int, const void*, const float*, const float*, Twist,
                                            const cx<float>*, cx<float>*, int, int, long, hipStream_t);
template void launch_sap<double, double>(const Geom&, int, const void*, const double*, const double*, Twist,
                                         const cx<double>*, cx<double>*, int, hipStream_t);
template void launch_sap<float, float>(const Geom&, int, const void*, const float*, const float*, Twist,
                                       const cx<float>*, cx<float>*, int, hipStream_t);
template void launch_sap<float, f16>(const Geom&, int, const void*, const float*, const float*, Twist,
                                        const cx<float>*, cx<float>*, int, hipStream_t);
template void launch_sap<float, bf16>(const Geom&, int, const void*, const float*, const float*, Twist,
                                                const cx<float>*, cx<float>*, int, hipStream_t);

// ---------------------------------------------------------------------------
// host TZYX lexicographic <-> block layout, K spinor fields (strides ldl, ldb
// complex), converted between FP64 and R on the way.  Bound by memory.  One
// workgroup per (block, field): the block's sites are read as whole runs along
// X, pass through LDS (12 components padded to 13) and are written as the
// block's one contiguous range, or the other way round; one thread per site
// moving its own 192 bytes reached half the rate (2.3 TB/s), and the conversion
// was another pass: the smoother's call on six BF16 fields at 48x24x24x24 spends
// 0.9 ms here instead of 2.9 ms.
namespace {
constexpr int LX = 13;  // components of a site in LDS, padded
// lexicographic site xof[j] and slot sof[j] of the block's j-th site (in
// lexicographic order inside the block)
__device__ __forceinline__ void block_sites(const Geom& g, int B, int s, int* xof, int* sof) {
  SiteNbr me;
  me_of(g, B, s, me);
  int x[4];
  for (int d = 0; d < 4; ++d) x[d] = me.bc[d] * g.b[d] + me.l[d];
  const int j = ((me.l[0] * g.b[1] + me.l[1]) * g.b[2] + me.l[2]) * g.b[3] + me.l[3];
  xof[j] = (int)lex_index(g, x);
  sof[j] = s;
}
}  // namespace
template <class L, class R>
__global__ void __launch_bounds__(256) k_spinor_from_lex(Geom g, const cx<L>* __restrict__ lex, long ldl,
                                                         cx<R>* __restrict__ out, long ldb) {
  extern __shared__ char smem_raw[];
  cx<R>* lds = reinterpret_cast<cx<R>*>(smem_raw);  // bs x LX
  __shared__ int xof[256], sof[256];
  const int B = blockIdx.x, s = threadIdx.x;
  lex += (long)blockIdx.y * ldl;
  out += (long)blockIdx.y * ldb + (long)B * g.bs * 12;
  block_sites(g, B, s, xof, sof);
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const int e = i * g.bs + s, j = e / 12, c = e - 12 * j;
    const cx<L> v = lex[(long)xof[j] * 12 + c];
    lds[sof[j] * LX + c] = mk<R>((R)v.re, (R)v.im);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const int e = i * g.bs + s, t = e / (12 * TILE), r = e - t * (12 * TILE);
    out[e] = lds[(t * TILE + (r % TILE)) * LX + r / TILE];
  }
}

template <class R>
__global__ void __launch_bounds__(256) k_spinor_to_lex(Geom g, const cx<R>* __restrict__ in, long ldb,
                                                       cx<double>* __restrict__ lex, long ldl) {
  extern __shared__ char smem_raw[];
  cx<R>* lds = reinterpret_cast<cx<R>*>(smem_raw);
  __shared__ int xof[256], sof[256];
  const int B = blockIdx.x, s = threadIdx.x;
  lex += (long)blockIdx.y * ldl;
  in += (long)blockIdx.y * ldb + (long)B * g.bs * 12;
  block_sites(g, B, s, xof, sof);
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const int e = i * g.bs + s, t = e / (12 * TILE), r = e - t * (12 * TILE);
    lds[(t * TILE + (r % TILE)) * LX + r / TILE] = in[e];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const int e = i * g.bs + s, j = e / 12, c = e - 12 * j;
    const cx<R> v = lds[sof[j] * LX + c];
    lex[(long)xof[j] * 12 + c] = mk<double>(v.re, v.im);
  }
}

template <class L, class R>
void launch_from_lex(const Geom& g, const cx<L>* lex, long ldl, cx<R>* out, long ldb, int K, hipStream_t st) {
  if (g.V > 0x7fffffffL) throw Error(INVALID_ARG, "lattice of 2^31 sites or more");
  hipLaunchKernelGGL((k_spinor_from_lex<L, R>), dim3(g.nblocks, K), dim3(g.bs), (size_t)LX * g.bs * sizeof(cx<R>), st,
                     g, lex, ldl, out, ldb);
}
template <class R>
void launch_to_lex(const Geom& g, const cx<R>* in, long ldb, cx<double>* lex, long ldl, int K, hipStream_t st) {
  if (g.V > 0x7fffffffL) throw Error(INVALID_ARG, "lattice of 2^31 sites or more");
  hipLaunchKernelGGL(k_spinor_to_lex<R>, dim3(g.nblocks, K), dim3(g.bs), (size_t)LX * g.bs * sizeof(cx<R>), st, g, in,
                     ldb, lex, ldl);
}
template void launch_from_lex<double, double>(const Geom&, const cx<double>*, long, cx<double>*, long, int, hipStream_t);
template void launch_from_lex<double, float>(const Geom&, const cx<double>*, long, cx<float>*, long, int, hipStream_t);
template void launch_from_lex<float, float>(const Geom&, const cx<float>*, long, cx<float>*, long, int, hipStream_t);
template void launch_to_lex<double>(const Geom&, const cx<double>*, long, cx<double>*, long, int, hipStream_t);
template void launch_to_lex<float>(const Geom&, const cx<float>*, long, cx<double>*, long, int, hipStream_t);

// ---------------------------------------------------------------------------
// clover term from the links: per site the six F_{mu nu} (mu<nu) from the four
// same-orientation plaquette leaves, then the two chirality blocks
// A_chi = (i c_sw / 2) sum_{mu<nu} sigma^chi_{mu nu} (x) F_{mu nu}; stored as
// H = (m0+4) + A, packed Hermitian.
//
// What bounds it is the links' way through the caches (8 GB of them at
// 48x24x24x24) and the latency of three dependent products.  One workgroup per
// 64 sites, two wavefronts that take three planes each, so that the plane and
// every loop over its links are uniform; one lane per site.  A lane holds a
// few 3x3 matrices in 242 registers (two wavefronts per SIMD, four workgroups
// per CU); one thread per site with all planes and both blocks of A kept 600
// reals in scratch memory.  F is anti-Hermitian: 9 reals per plane go through
// LDS to the second half, where a thread forms one packed entry of 8 sites in
// the order in which they are stored.  48x24x24x24: 4370 -> 690 us (six
// wavefronts of one plane each: 810 us, since six of eight slots are used;
// three wavefronts per SIMD spill 48 registers: 1060 us).
struct Mat3 {
  cx<double> m[9];
};

// link mu of the site a steps along mu0 and b steps along nu0 from `me`
// (|a|, |b| <= 1)
__device__ __forceinline__ Mat3 leaf_link(const cx<double>* U, const Geom& g, const SiteNbr& me, int mu0, int a,
                                          int nu0, int b, int mu) {
  SiteNbr y = me;
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const int st = d == mu0 ? a : d == nu0 ? b : 0;
    int l = y.l[d] + st, c = y.bc[d];
    if (l == g.b[d]) {
      l = 0;
      c = c + 1 == g.nb[d] ? 0 : c + 1;
    } else if (l < 0) {
      l = g.b[d] - 1;
      c = c == 0 ? g.nb[d] - 1 : c - 1;
    }
    y.l[d] = l;
    y.bc[d] = c;
  }
  const cx<double>* p = U + fidx(g, block_index(g, y.bc), local_slot(g, y.l), 36) + (long)mu * 9 * TILE;
  Mat3 r;
#pragma unroll
  for (int k = 0; k < 9; ++k) r.m[k] = p[k * TILE];
  return r;
}
// a b, a b^dag (DB) or a^dag b (DA)
template <bool DA, bool DB>
__device__ __forceinline__ Mat3 mul(const Mat3& a, const Mat3& b) {
  Mat3 r;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      cx<double> acc = mk(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < 3; ++k)
        cmac(acc, DA ? conj(a.m[3 * k + i]) : a.m[3 * i + k], DB ? conj(b.m[3 * j + k]) : b.m[3 * k + j]);
      r.m[3 * i + j] = acc;
    }
  return r;
}

// sigma^chi_{mu nu} for mu<nu, pair index p (01,02,03,12,13,23), 2x2 per chirality
__constant__ double c_sigma[6][2][4][2];

// The four leaves of one orientation, Q = L1 + L2 + L3 + L4, with
//   L1 = U_mu(x) U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
//   L2 = U_nu(x) U_mu(x-mu+nu)^dag U_nu(x-mu)^dag U_mu(x-mu)
//   L3 = U_mu(x-mu)^dag U_nu(x-mu-nu)^dag U_mu(x-mu-nu) U_nu(x-nu)
//   L4 = U_nu(x-nu)^dag U_mu(x-nu) U_nu(x+mu-nu) U_mu(x)^dag,
// enter only through Q - Q^dag, which is A - A^dag with
//   A = U_mu(x) [S0 - S1] + U_mu(x-mu)^dag [S2 - S3],
//   S0 = U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag        S1 = U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu)
//   S2 = U_nu(x-mu-nu)^dag U_mu(x-mu-nu) U_nu(x-nu)   S3 = U_nu(x-mu) U_mu(x-mu+nu) U_nu(x)^dag
// (ten products and 14 links instead of 12 and 16).
__global__ void __launch_bounds__(128) k_clover(Geom g, const cx<double>* __restrict__ U, double csw, double diag,
                                                double* __restrict__ H) {
  // F of each plane: Im diagonal, then (re, im) of 01, 02, 12; rows padded
  // against bank conflicts (8 sites of 4 consecutive rows cover the banks)
  __shared__ double fs[6][9][72];
  const int lane = threadIdx.x & 63;
  // each XCD takes a contiguous range of sites: a site's links serve its
  // neighbours' leaves from the same L2
  const long wg = xcd_remap(blockIdx.x, gridDim.x);
  const long gid = wg * 64 + lane;
#pragma unroll 1
  for (int p = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); p < 6; p += 2) {
    if (gid >= g.V) break;
    const int mu = p < 3 ? 0 : p < 5 ? 1 : 2, nu = p < 3 ? p + 1 : p < 5 ? p - 1 : 3;
    const int B = (int)(gid / g.bs), s = (int)(gid - (long)B * g.bs);
    SiteNbr me;
    me_of(g, B, s, me);
    auto link = [&](int a, int b, int d) { return leaf_link(U, g, me, mu, a, nu, b, d ? nu : mu); };
    Mat3 S, A;
    // one staple at a time (the loop stays rolled): at most four matrices live
#pragma unroll 1
    for (int t = 0; t < g.ndir; ++t) {
      Mat3 T;
      switch (t) {
        case 0: T = mul<false, true>(mul<false, true>(link(1, 0, 1), link(0, 1, 0)), link(0, 0, 1)); break;
        case 1: T = mul<true, false>(mul<false, false>(link(0, -1, 0), link(1, -1, 1)), link(0, -1, 1)); break;
        case 2: T = mul<true, false>(link(-1, -1, 1), mul<false, false>(link(-1, -1, 0), link(0, -1, 1))); break;
        default: T = mul<false, true>(mul<false, false>(link(-1, 0, 1), link(-1, 1, 0)), link(0, 0, 1)); break;
      }
#pragma unroll
      for (int k = 0; k < 9; ++k) S.m[k] = t & 1 ? S.m[k] - T.m[k] : T.m[k];
      if (t == 1) A = mul<false, false>(link(0, 0, 0), S);
      if (t == 3) {
        T = mul<true, false>(link(-1, 0, 0), S);
#pragma unroll
        for (int k = 0; k < 9; ++k) A.m[k] += T.m[k];
      }
    }
    // F = (A - A^dag) / 8
#pragma unroll
    for (int a = 0; a < 3; ++a) fs[p][a][lane] = 0.25 * A.m[4 * a].im;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int a = q == 2 ? 1 : 0, b = q == 0 ? 1 : 2;
      fs[p][3 + 2 * q][lane] = 0.125 * (A.m[3 * a + b].re - A.m[3 * b + a].re);
      fs[p][4 + 2 * q][lane] = 0.125 * (A.m[3 * a + b].im + A.m[3 * b + a].im);
    }
  }
  __syncthreads();
  // thread = (packed entry kk of a block, site in a tile): its entry (i, j) and
  // the coefficients (i c_sw / 2) sigma of the six planes are fixed
  for (int role = threadIdx.x; role < 36 * 8; role += 128) {
    const int kk = role >> 3, st = role & 7;
    int i = kk, j = kk;
    if (kk >= 6) {  // off-diagonal pair number (kk - 6) / 2, row-major i < j
      int q = (kk - 6) >> 1;
      i = 0;
      while (q >= 5 - i) {
        q -= 5 - i;
        ++i;
      }
      j = i + 1 + q;
    }
    const int s1 = i >= 3, s2 = j >= 3, a = i - 3 * s1, b = j - 3 * s2;
    // F[a][b]: real part from row fr (zero on the diagonal), imaginary part from
    // row fi; F[b][a] = -conj(F[a][b])
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    const int fi = a == b ? a : 4 + 2 * (lo + hi - 1), fr = a == b ? a : fi - 1;
    const double sr = a == b ? 0.0 : a < b ? 1.0 : -1.0;
    const bool im = kk >= 6 && (kk & 1);
    double* hp = H + wg * 64 * 72 + st;
    const int ntile = (int)(g.V - wg * 64 < 64 ? (g.V - wg * 64) >> 3 : 8);
    for (int c = 0; c < 2; ++c) {
      // the wanted part of coef * F is p fr + q fi
      double p_[6], q_[6];
#pragma unroll
      for (int pl = 0; pl < 6; ++pl) {
        const double cr = -0.5 * csw * c_sigma[pl][c][2 * s1 + s2][1], ci = 0.5 * csw * c_sigma[pl][c][2 * s1 + s2][0];
        p_[pl] = sr * (im ? ci : cr);
        q_[pl] = im ? cr : -ci;
      }
#pragma unroll 2
      for (int tile = 0; tile < ntile; ++tile) {
        double v = kk < 6 ? diag : 0.0;
#pragma unroll
        for (int pl = 0; pl < 6; ++pl)
          v += p_[pl] * fs[pl][fr][8 * tile + st] + q_[pl] * fs[pl][fi][8 * tile + st];
        hp[(long)tile * 576 + (36 * c + kk) * 8] = v;
      }
    }
  }
}

void set_sigma_table(const double* tab /* [6][2][4][2] */) {
  HIP_CHECK(hipMemcpyToSymbol(HIP_SYMBOL(c_sigma), tab, sizeof(double) * 6 * 2 * 4 * 2));
}

void launch_clover(const Geom& g, const cx<double>* U, double csw, double diag, double* H, hipStream_t st) {
  hipLaunchKernelGGL(k_clover, dim3((unsigned)((g.V + 63) / 64)), dim3(128), 0, st, g, U, csw, diag, H);
}

// user-supplied clover term [V][2][6][6] (lexicographic) -> packed H = diag + A
__global__ void k_clover_from_lex(Geom g, const cx<double>* __restrict__ lex, double diag, double* __restrict__ H) {
  long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= g.V) return;
  int B = (int)(gid / g.bs), s = (int)(gid - (long)B * g.bs);
  int x[4];
  site_coords(g, B, s, x);
  long li = lex_index(g, x);
  double* hp = H + fidx(g, B, s, 72);
  for (int c = 0; c < 2; ++c) {
    const cx<double>* a = lex + (li * 2 + c) * 36;
    double* h = hp + 36L * c * TILE;
    for (int i = 0; i < 6; ++i) h[(long)i * TILE] = diag + a[6 * i + i].re;
    for (int i = 0; i < 6; ++i)
      for (int j = i + 1; j < 6; ++j) {
        int k = 6 + 2 * herm_idx(i, j);
        cx<double> v = 0.5 * (a[6 * i + j] + conj(a[6 * j + i]));
        h[(long)k * TILE] = v.re;
        h[(long)(k + 1) * TILE] = v.im;
      }
  }
}
void launch_clover_from_lex(const Geom& g, const cx<double>* lex, double diag, double* H, hipStream_t st) {
  hipLaunchKernelGGL(k_clover_from_lex, dim3((g.V + 127) / 128), dim3(128), 0, st, g, lex, diag, H);
}

// packed H (without m0+4) back to [V][2][6][6] lexicographic
__global__ void k_clover_to_lex(Geom g, const double* __restrict__ H, double diag, cx<double>* __restrict__ lex) {
  long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= g.V) return;
  int B = (int)(gid / g.bs), s = (int)(gid - (long)B * g.bs);
  int x[4];
  site_coords(g, B, s, x);
  long li = lex_index(g, x);
  const double* hp = H + fidx(g, B, s, 72);
  for (int c = 0; c < 2; ++c) {
    cx<double>* a = lex + (li * 2 + c) * 36;
    const double* h = hp + 36L * c * TILE;
    for (int i = 0; i < 6; ++i) a[6 * i + i] = mk(h[(long)i * TILE] - diag, 0.0);
    for (int i = 0; i < 6; ++i)
      for (int j = i + 1; j < 6; ++j) {
        int k = 6 + 2 * herm_idx(i, j);
        cx<double> v = mk(h[(long)k * TILE], h[(long)(k + 1) * TILE]);
        a[6 * i + j] = v;
        a[6 * j + i] = conj(v);
      }
  }
}
void launch_clover_to_lex(const Geom& g, const double* H, double diag, cx<double>* lex, hipStream_t st) {
  hipLaunchKernelGGL(k_clover_to_lex, dim3((g.V + 127) / 128), dim3(128), 0, st, g, H, diag, lex);
}

// links [V][4][3][3] lexicographic -> block layout FP64
__global__ void k_links_from_lex(Geom g, const cx<double>* __restrict__ lex, cx<double>* __restrict__ U,
                                 LinkPhases ph) {
  long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= g.V) return;
  int B = (int)(gid / g.bs), s = (int)(gid - (long)B * g.bs);
  int x[4];
  site_coords(g, B, s, x);
  long li = lex_index(g, x);
  for (int mu = 0; mu < 4; ++mu) {
    const bool edge = x[mu] == g.L[mu] - 1;
    const cx<double> f = edge ? mk(ph.re[mu], ph.im[mu]) : mk(1.0, 0.0);
    for (int k = 0; k < 9; ++k) {
      const cx<double> v = lex[(li * 4 + mu) * 9 + k];
      U[fidx(g, B, s, 36) + (long)(mu * 9 + k) * TILE] = edge ? f * v : v;
    }
  }
}
void launch_links_from_lex(const Geom& g, const cx<double>* lex, cx<double>* U, const LinkPhases& ph,
                           hipStream_t st) {
  hipLaunchKernelGGL(k_links_from_lex, dim3((g.V + 255) / 256), dim3(256), 0, st, g, lex, U, ph);
}

// twisted boundary conditions psi(x + L_mu e_mu) = e^{i theta_mu} psi(x) as a
// phase on the links that cross the boundary (forward hop from x_mu = L_mu - 1
// and, through U^dag, the backward hop from x_mu = 0)
__global__ void k_link_phase(Geom g, cx<double>* __restrict__ U, LinkPhases ph) {
  long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= g.V) return;
  int B = (int)(gid / g.bs), s = (int)(gid - (long)B * g.bs);
  int x[4];
  site_coords(g, B, s, x);
  for (int mu = 0; mu < 4; ++mu) {
    if (x[mu] != g.L[mu] - 1) continue;
    const cx<double> f = mk(ph.re[mu], ph.im[mu]);
    for (int k = 0; k < 9; ++k) {
      cx<double>& v = U[fidx(g, B, s, 36) + (long)(mu * 9 + k) * TILE];
      v = f * v;
    }
  }
}
void launch_link_phase(const Geom& g, cx<double>* U, const LinkPhases& ph, hipStream_t st) {
  hipLaunchKernelGGL(k_link_phase, dim3((g.V + 255) / 256), dim3(256), 0, st, g, U, ph);
}

// out += i rho Gamma5 in on the odd sites: the twist of the odd sites raised
// by rho over that of the even sites (FP64 fine fields)
__global__ void k_odd_twist_add(Geom g, const cx<double>* __restrict__ in, cx<double>* __restrict__ out, double rho) {
  long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long)g.nblocks * g.half) return;
  int B = (int)(gid / g.half), s = g.half + (int)(gid - (long)B * g.half);
  const long o = fidx(g, B, s, 12);
  for (int c = 0; c < 12; ++c) {
    const double t = c < 6 ? -rho : rho;  // Gamma5 = diag(-1, -1, 1, 1) in spin
    const cx<double> v = in[o + (long)c * TILE];
    cx<double> w = out[o + (long)c * TILE];
    w.re -= t * v.im;
    w.im += t * v.re;
    out[o + (long)c * TILE] = w;
  }
}
void launch_odd_twist_add(const Geom& g, const cx<double>* in, cx<double>* out, double rho, hipStream_t st) {
  const long n = (long)g.nblocks * g.half;
  hipLaunchKernelGGL(k_odd_twist_add, dim3((n + 255) / 256), dim3(256), 0, st, g, in, out, rho);
}

// x = 0 on the even sites (FP64 fine field)
__global__ void k_zero_even(Geom g, cx<double>* __restrict__ x) {
  long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long)g.nblocks * g.half) return;
  int B = (int)(gid / g.half), s = (int)(gid - (long)B * g.half);
  const long o = fidx(g, B, s, 12);
  for (int c = 0; c < 12; ++c) x[o + (long)c * TILE] = mk(0.0, 0.0);
}
void launch_zero_even(const Geom& g, cx<double>* x, hipStream_t st) {
  const long n = (long)g.nblocks * g.half;
  hipLaunchKernelGGL(k_zero_even, dim3((n + 255) / 256), dim3(256), 0, st, g, x);
}

// ---------------------------------------------------------------------------
// odd-site inverse factor M_chi = (H_chi^2 + tw^2)^{-1} (Hermitian positive
// definite), stored packed like H.  One thread per (odd site, chirality): the
// packed G = H^2 + tw^2 (36 reals) is inverted in place by the Hermitian
// Gauss-Jordan sweep (no pivoting: G is positive definite), so H and G are all
// that a thread holds and both stay in registers; a Cholesky factorisation with
// separate full matrices kept 600 reals in scratch memory.  Bound by memory:
// 48x24x24x24 402 -> 67 us, 5.7 TB/s of its 382 MB.
// packed index of the real part of entry (i < j)
__device__ constexpr int pk(int i, int j) { return 6 + 2 * (5 * i - (i * (i - 1)) / 2 + (j - i - 1)); }
__device__ __forceinline__ cx<double> pget(const double (&h)[36], int i, int j) {
  if (i == j) return mk(h[i], 0.0);
  return i < j ? mk(h[pk(i, j)], h[pk(i, j) + 1]) : mk(h[pk(j, i)], -h[pk(j, i) + 1]);
}
__global__ void __launch_bounds__(128) k_odd_inverse(Geom g, const double* __restrict__ H, double tw,
                                                     double* __restrict__ M) {
  const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  // (tile of 8 odd sites, chirality, site in the tile): 8 consecutive threads
  // read 64 contiguous bytes of every packed entry
  const long tl = gid >> 4;
  const int c = (int)(gid >> 3) & 1;
  const long odd = tl * 8 + (gid & 7);
  if (odd >= (long)g.nblocks * g.half) return;
  const int B = (int)(odd / g.half), io = (int)(odd - (long)B * g.half);
  const double* hc = H + fidx(g, B, g.half + io, 72) + 36L * c * TILE;
  double h[36], G[36];
#pragma unroll
  for (int k = 0; k < 36; ++k) h[k] = hc[k * TILE];
#pragma unroll
  for (int i = 0; i < 6; ++i)
#pragma unroll
    for (int j = i; j < 6; ++j) {
      cx<double> acc = mk(i == j ? tw * tw : 0.0, 0.0);
#pragma unroll
      for (int k = 0; k < 6; ++k) cmac(acc, pget(h, i, k), pget(h, k, j));
      if (i == j) {
        G[i] = acc.re;
      } else {
        G[pk(i, j)] = acc.re;
        G[pk(i, j) + 1] = acc.im;
      }
    }
  // sweep of every pivot: G_kk -> -1/d, G_ik -> G_ik/d, G_ij -> G_ij - G_ik G_kj/d;
  // after all six the matrix is -G^{-1}
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const double d = 1.0 / G[k];
    cx<double> col[6];  // G_ik
#pragma unroll
    for (int i = 0; i < 6; ++i) col[i] = pget(G, i, k);
#pragma unroll
    for (int i = 0; i < 6; ++i)
#pragma unroll
      for (int j = i; j < 6; ++j) {
        if (i == k || j == k) continue;
        // G_ik G_kj / d = col_i conj(col_j) / d
        const cx<double> t = col[i] * conj(d * col[j]);
        if (i == j) {
          G[i] -= d * (col[i].re * col[i].re + col[i].im * col[i].im);
        } else {
          G[pk(i, j)] -= t.re;
          G[pk(i, j) + 1] -= t.im;
        }
      }
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      if (i == k) continue;
      const cx<double> t = d * col[i];
      if (i < k) {
        G[pk(i, k)] = t.re;
        G[pk(i, k) + 1] = t.im;
      } else {
        G[pk(k, i)] = t.re;
        G[pk(k, i) + 1] = -t.im;
      }
    }
    G[k] = -d;
  }
  double* mp = M + oidx(g, B, io, 72) + 36L * c * TILE;
#pragma unroll
  for (int k = 0; k < 36; ++k) mp[k * TILE] = -G[k];
}
void launch_odd_inverse(const Geom& g, const double* H, double tw, double* M, hipStream_t st) {
  const long n = 2 * (long)g.nblocks * g.half;
  hipLaunchKernelGGL(k_odd_inverse, dim3((unsigned)((n + 127) / 128)), dim3(128), 0, st, g, H, tw, M);
}

// ---------------------------------------------------------------------------
// restriction P^dag on the fine level: one workgroup per block (= aggregate),
// one thread per slot; output r_c[site][s*Nv + i].
// One thread per slot (threads past the block's slots contribute zero), four test
// vectors at a time: their 16 FP64 sums go over the wavefront by a transposing
// butterfly and over the wavefronts in LDS.  Few blocks: groups of vectors in
// workgroups of their own, or 32 blocks keep 32 CUs busy (16 vectors, 8x8x8x16:
// 56 -> 6.5 us).
template <class R>
__global__ void __launch_bounds__(256) k_restrict_fine(Geom g, int Nv, const cx<R>* __restrict__ Q, long vstride,
                                                       const cx<R>* __restrict__ r, const int* __restrict__ f2c,
                                                       cx<R>* __restrict__ rc) {
  constexpr int II = 4, NVAL = 4 * II;
  __shared__ double red[2][4][NVAL];
  const int B = blockIdx.x, s = threadIdx.x, lane = s & 63, wv = s >> 6, nw = blockDim.x >> 6;
  const bool live = s < g.bs;
  const long base = fidx(g, B, live ? s : 0, 12);
  const int site = f2c[B];
  cx<R> rv[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    rv[c] = r[base + (long)c * TILE];
    if (!live) rv[c] = mk<R>(0, 0);
  }
  int p = 0;
  for (int i0 = II * blockIdx.y; i0 < Nv; i0 += II * gridDim.y, p ^= 1) {
    double acc[NVAL];
#pragma unroll
    for (int v = 0; v < NVAL; ++v) acc[v] = 0.0;
#pragma unroll
    for (int ii = 0; ii < II; ++ii) {
      const cx<R>* q = Q + (long)min(i0 + ii, Nv - 1) * vstride + base;  // sums past Nv unused
      cx<R> qv[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        qv[c] = q[(long)c * TILE];
        if (!live) qv[c] = mk<R>(0, 0);
      }
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        const int v = 4 * ii + 2 * (c / 6);
        acc[v] += (double)qv[c].re * rv[c].re + (double)qv[c].im * rv[c].im;
        acc[v + 1] += (double)qv[c].re * rv[c].im - (double)qv[c].im * rv[c].re;
      }
    }
    const double tot = wave_transpose_sum<NVAL>(acc, lane);
    if (lane < NVAL) red[p][wv][lane] = tot;
    __syncthreads();
    const int i = i0 + (s >> 2);
    if (s < NVAL && i < Nv) {
      double sum = 0.0;
      for (int v = 0; v < nw; ++v) sum += red[p][v][s];
      reinterpret_cast<R*>(rc + (long)site * 2 * Nv + ((s >> 1) & 1) * Nv + i)[s & 1] = (R)sum;
    }
  }
}

template <class R>
void launch_restrict_fine(const Geom& g, int Nv, const cx<R>* Q, long vstride, const cx<R>* r, const int* f2c,
                          cx<R>* rc, hipStream_t st) {
  // from 1024 blocks on a workgroup reads r once for all vectors (2048 blocks of 256
  // sites, 16 vectors: 162 us, 5 TB/s)
  const int ny = g.nblocks >= 1024 ? 1 : (Nv + 3) / 4;
  hipLaunchKernelGGL(k_restrict_fine<R>, dim3(g.nblocks, ny), dim3((g.bs + 63) / 64 * 64), 0, st, g, Nv, Q, vstride, r,
                     f2c, rc);
}
template void launch_restrict_fine<double>(const Geom&, int, const cx<double>*, long, const cx<double>*,
                                           const int*, cx<double>*, hipStream_t);
template void launch_restrict_fine<float>(const Geom&, int, const cx<float>*, long, const cx<float>*, const int*,
                                          cx<float>*, hipStream_t);

// prolongation P: x (+)= sum_i Q_i e_c(s(comp)*Nv + i)
template <class R>
__global__ void __launch_bounds__(256) k_prolong_fine(Geom g, int Nv, const cx<R>* __restrict__ Q, long vstride,
                                                      const cx<R>* __restrict__ ec, const int* __restrict__ f2c,
                                                      cx<R>* __restrict__ x, int accumulate) {
  long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= g.V) return;
  int B = (int)(gid / g.bs), s = (int)(gid - (long)B * g.bs);
  const cx<R>* e = ec + (long)f2c[B] * 2 * Nv;
  cx<R> acc[12];
  if (accumulate) load_spinor(x, g, B, s, acc);
  else
    for (int c = 0; c < 12; ++c) acc[c] = mk<R>(0, 0);
  long base = fidx(g, B, s, 12);
  for (int i = 0; i < Nv; ++i) {
    cx<R> e0 = e[i], e1 = e[Nv + i];
    const cx<R>* q = Q + (long)i * vstride + base;
#pragma unroll
    for (int c = 0; c < 6; ++c) cmac(acc[c], q[(long)c * TILE], e0);
#pragma unroll
    for (int c = 6; c < 12; ++c) cmac(acc[c], q[(long)c * TILE], e1);
  }
  store_spinor(x, g, B, s, acc);
}
template <class R>
void launch_prolong_fine(const Geom& g, int Nv, const cx<R>* Q, long vstride, const cx<R>* ec, const int* f2c,
                         cx<R>* x, int accumulate, hipStream_t st) {
  hipLaunchKernelGGL(k_prolong_fine<R>, dim3((g.V + 255) / 256), dim3(256), 0, st, g, Nv, Q, vstride, ec, f2c, x,
                     accumulate);
}
template void launch_prolong_fine<double>(const Geom&, int, const cx<double>*, long, const cx<double>*, const int*,
                                          cx<double>*, int, hipStream_t);
template void launch_prolong_fine<float>(const Geom&, int, const cx<float>*, long, const cx<float>*, const int*,
                                         cx<float>*, int, hipStream_t);

// K-column restriction: one thread per slot (threads past the block's slots
// contribute zero), columns in groups of KC whose inputs stay in registers, test
// vectors in groups of II, so Q is read once per group of columns.  The 4 II KC
// values (vector, column, half, re/im) of a group, padded to a power of two,
// are summed over the wavefront by a transposing butterfly and over the
// wavefronts in LDS in fixed order.
template <int N>
constexpr int pow2_ceil() {
  int p = 1;
  while (p < N) p *= 2;
  return p;
}
template <class R, int KC, int II>
__global__ void __launch_bounds__(256) k_restrict_fine_m(Geom g, int Nv, const cx<R>* __restrict__ Q, long vstride,
                                                         const cx<R>* __restrict__ r, long rld, int K,
                                                         const int* __restrict__ f2c, cx<R>* __restrict__ rc,
                                                         long cld) {
  constexpr int NV0 = 4 * II * KC, NVAL = pow2_ceil<NV0>();
  __shared__ R red[4][NVAL];
  const int B = blockIdx.x, s = threadIdx.x, lane = s & 63, wv = s >> 6, nw = blockDim.x >> 6;
  const bool live = s < g.bs;
  const long site = f2c[B];
  const long base = live ? fidx(g, B, s, 12) : 0;
  for (int k0 = 0; k0 < K; k0 += KC) {
    cx<R> rv[KC][12];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk)
#pragma unroll
      for (int c = 0; c < 12; ++c)
        rv[kk][c] = live && k0 + kk < K ? r[(long)(k0 + kk) * rld + base + (long)c * TILE] : mk<R>(0, 0);
    for (int i0 = 0; i0 < Nv; i0 += II) {
      R acc[NVAL];
#pragma unroll
      for (int v = 0; v < NVAL; ++v) acc[v] = R(0);
#pragma unroll
      for (int ii = 0; ii < II; ++ii) {
        const int i = i0 + ii;
        if (i < Nv && live) {
          cx<R> q[12];
#pragma unroll
          for (int c = 0; c < 12; ++c) q[c] = Q[(long)i * vstride + base + (long)c * TILE];
#pragma unroll
          for (int kk = 0; kk < KC; ++kk)
#pragma unroll
            for (int c = 0; c < 12; ++c) {
              const int v = ((ii * KC + kk) * 2 + c / 6) * 2;
              acc[v] += q[c].re * rv[kk][c].re + q[c].im * rv[kk][c].im;
              acc[v + 1] += q[c].re * rv[kk][c].im - q[c].im * rv[kk][c].re;
            }
        }
      }
      const R tot = wave_transpose_sum<NVAL>(acc, lane);
      if (lane < NVAL) red[wv][lane] = tot;
      __syncthreads();
      if (s < NV0) {
        R sum = R(0);
        for (int w = 0; w < nw; ++w) sum += red[w][s];
        const int p = s & 1, h = (s >> 1) & 1, kk = (s >> 2) % KC, ii = (s >> 2) / KC;
        const int i = i0 + ii, k = k0 + kk;
        if (i < Nv && k < K) reinterpret_cast<R*>(rc + (long)k * cld + site * 2 * Nv + h * Nv + i)[p] = sum;
      }
      __syncthreads();
    }
  }
}
template <class R>
void launch_restrict_fine_m(const Geom& g, int Nv, const cx<R>* Q, long vstride, const cx<R>* r, long rld, int K,
                            const int* f2c, cx<R>* rc, long cld, hipStream_t st) {
  const dim3 grid(g.nblocks), blk(((g.bs + 63) / 64) * 64);
  if (K == 1)
    hipLaunchKernelGGL((k_restrict_fine_m<R, 1, 4>), grid, blk, 0, st, g, Nv, Q, vstride, r, rld, K, f2c, rc, cld);
  else if (K == 2 || sizeof(R) == 8)
    hipLaunchKernelGGL((k_restrict_fine_m<R, 2, 4>), grid, blk, 0, st, g, Nv, Q, vstride, r, rld, K, f2c, rc, cld);
  else if (K == 5 || K == 6)
    hipLaunchKernelGGL((k_restrict_fine_m<R, 6, 1>), grid, blk, 0, st, g, Nv, Q, vstride, r, rld, K, f2c, rc, cld);
  else
    hipLaunchKernelGGL((k_restrict_fine_m<R, 4, 4>), grid, blk, 0, st, g, Nv, Q, vstride, r, rld, K, f2c, rc, cld);
}
template void launch_restrict_fine_m<double>(const Geom&, int, const cx<double>*, long, const cx<double>*, long, int,
                                             const int*, cx<double>*, long, hipStream_t);
template void launch_restrict_fine_m<float>(const Geom&, int, const cx<float>*, long, const cx<float>*, long, int,
                                            const int*, cx<float>*, long, hipStream_t);

// K-column prolongation: x_k (+)= sum_i Q_i e_k, one thread per site, columns in
// groups of KC accumulated in registers (Q read once per group)
template <class R, int KC>
__global__ void __launch_bounds__(256) k_prolong_fine_m(Geom g, int Nv, const cx<R>* __restrict__ Q, long vstride,
                                                        const cx<R>* __restrict__ ec, long cld, int K,
                                                        const int* __restrict__ f2c, cx<R>* __restrict__ x, long xld,
                                                        int accumulate) {
  const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= g.V) return;
  const int B = (int)(gid / g.bs), s = (int)(gid - (long)B * g.bs);
  const cx<R>* e = ec + (long)f2c[B] * 2 * Nv;
  const long base = fidx(g, B, s, 12);
  for (int k0 = 0; k0 < K; k0 += KC) {
    cx<R> acc[KC][12];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk)
#pragma unroll
      for (int c = 0; c < 12; ++c)
        acc[kk][c] = accumulate && k0 + kk < K ? x[(long)(k0 + kk) * xld + base + (long)c * TILE] : mk<R>(0, 0);
    for (int i = 0; i < Nv; ++i) {
      cx<R> q[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) q[c] = Q[(long)i * vstride + base + (long)c * TILE];
#pragma unroll
      for (int kk = 0; kk < KC; ++kk) {
        if (k0 + kk >= K) continue;
        const cx<R> e0 = e[(long)(k0 + kk) * cld + i], e1 = e[(long)(k0 + kk) * cld + Nv + i];
#pragma unroll
        for (int c = 0; c < 6; ++c) cmac(acc[kk][c], q[c], e0);
#pragma unroll
        for (int c = 6; c < 12; ++c) cmac(acc[kk][c], q[c], e1);
      }
    }
#pragma unroll
    for (int kk = 0; kk < KC; ++kk)
      if (k0 + kk < K)
#pragma unroll
        for (int c = 0; c < 12; ++c) x[(long)(k0 + kk) * xld + base + (long)c * TILE] = acc[kk][c];
  }
}
template <class R>
void launch_prolong_fine_m(const Geom& g, int Nv, const cx<R>* Q, long vstride, const cx<R>* ec, long cld, int K,
                           const int* f2c, cx<R>* x, long xld, int accumulate, hipStream_t st) {
  const dim3 grid((unsigned)((g.V + 255) / 256)), blk(256);
  if (K == 1)
    hipLaunchKernelGGL((k_prolong_fine_m<R, 1>), grid, blk, 0, st, g, Nv, Q, vstride, ec, cld, K, f2c, x, xld, accumulate);
  else if (K == 2 || sizeof(R) == 8)
    hipLaunchKernelGGL((k_prolong_fine_m<R, 2>), grid, blk, 0, st, g, Nv, Q, vstride, ec, cld, K, f2c, x, xld, accumulate);
  else if (K == 5 || K == 6)
    hipLaunchKernelGGL((k_prolong_fine_m<R, 6>), grid, blk, 0, st, g, Nv, Q, vstride, ec, cld, K, f2c, x, xld, accumulate);
  else
    hipLaunchKernelGGL((k_prolong_fine_m<R, 4>), grid, blk, 0, st, g, Nv, Q, vstride, ec, cld, K, f2c, x, xld, accumulate);
}
template void launch_prolong_fine_m<double>(const Geom&, int, const cx<double>*, long, const cx<double>*, long, int,
                                            const int*, cx<double>*, long, int, hipStream_t);
template void launch_prolong_fine_m<float>(const Geom&, int, const cx<float>*, long, const cx<float>*, long, int,
                                           const int*, cx<float>*, long, int, hipStream_t);

// ---------------------------------------------------------------------------
// Galerkin assembly of the first coarse operator on the matrix cores.  One
// workgroup (4 wavefronts) per (block, kind), each kind a sum over a list of
// sites x of rank-6 products
//   C[(i,a),(j,b)] += sum_{c in half a} conj(Q_i(x)_c) Y_(j,b)(x)_c,
// with Y_(j,b) a right factor applied to the chirality-b half of Q_j:
//   kind 0 (self block S, every site):  Y = H(x) P_b Q_j(x)
//   kind 1 (internal links X, every site):
//       Y = sum_{mu: x+mu in block} -1/2 (1-g_mu) U_mu(x) P_b Q_j(x+mu)
//   kind 2+mu (forward block mu, sites on the upper mu face):
//       Y = -1/2 (1-g_mu) U_mu(x) P_b Q_j(x+mu)
// S goes to the self block, X to Xs for the fix-up S += X + Gamma5 X^dag Gamma5
// (k_self_fixup), the face kinds to the forward blocks; output blocks are
// column-major (element (k,l) at l*n + k).
// The complex products run as real ones on 16x16x4 MFMA (FP64 for an FP64 Q,
// FP32 for an FP32 Q): rows (i,a) are padded to 32 per half, wavefront w owning
// half a = w/2 and rows 16(w%2)..+15; the contraction index is (x, c in half a,
// re/im); columns (j,b) go in groups of 16 with a real and an imaginary tile
// (conj(q) y = (q.re y.re + q.im y.im) + i (q.re y.im - q.im y.re)).  CS sites
// at a time are staged in LDS: Q(x) with H(x) or U(x), then Y, built in the
// product's precision by one thread per (site, column).
namespace {
typedef double v4d_a __attribute__((ext_vector_type(4)));
typedef float v4f_a __attribute__((ext_vector_type(4)));
// lane L supplies A[L%16][L/16] and B[L/16][L%16]; element e of the
// accumulator holds D[row(L, e)][L%16], with row = L/16 + 4e for FP64 and
// 4(L/16) + e for FP32 (measured on gfx950)
template <class T> struct mfma_k4;
template <> struct mfma_k4<double> {
  typedef v4d_a acc;
  static __device__ __forceinline__ acc step(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int e) { return (lane >> 4) + 4 * e; }
};
template <> struct mfma_k4<float> {
  typedef v4f_a acc;
  static __device__ __forceinline__ acc step(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int e) { return 4 * (lane >> 4) + e; }
};

// slot of face site f of the upper mu face (the other coordinates in TZYX order)
__device__ __forceinline__ int face_slot(const Geom& g, int mu, int f) {
  int l[4];
  for (int d = 3; d >= 0; --d) {
    if (d == mu) {
      l[d] = g.b[d] - 1;
    } else {
      l[d] = f % g.b[d];
      f /= g.b[d];
    }
  }
  return local_slot(g, l);
}

// y += -1/2 (1-g_MU) U psi, psi = the chirality-HB half p6 of a spinor (other
// half zero), U = up[0..8]; arithmetic in T
template <int MU, int HB, class RQ, class T>
__device__ __forceinline__ void half_hop(const cx<RQ> p6[6], const cx<T>* up, cx<T> y[12]) {
  cx<T> psi[12], u[9];
#pragma unroll
  for (int c = 0; c < 12; ++c) psi[c] = mk<T>(0, 0);
#pragma unroll
  for (int c = 0; c < 6; ++c) psi[6 * HB + c] = mk<T>((T)p6[c].re, (T)p6[c].im);
#pragma unroll
  for (int k = 0; k < 9; ++k) u[k] = up[k];
  hop_accum_t<0, MU>(psi, u, y);
}
template <int MU, class RQ, class T>
__device__ __forceinline__ void half_hop(int hb, const cx<RQ> p6[6], const cx<T>* up, cx<T> y[12]) {
  if (hb) half_hop<MU, 1>(p6, up, y);
  else half_hop<MU, 0>(p6, up, y);
}
}  // namespace

template <class RQ, class T, int CS, int NG>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 4, 8)))
k_assemble_fine(Geom g, int Nv, const cx<double>* __restrict__ U, const double* __restrict__ H, double dtw,
                const cx<RQ>* __restrict__ Q, long qstride, const int* __restrict__ f2c, cx<double>* __restrict__ Dc,
                cx<double>* __restrict__ Xs) {
  using MF = mfma_k4<T>;
  using acc_t = typename MF::acc;
  constexpr int NC = 16 * NG;         // padded complex columns
  __shared__ cx<T> qs[CS][12][32];    // Q_i(x)_c, rows i padded to 32
  __shared__ cx<T> ys[CS][12][NC];    // Y_col(x)_c
  __shared__ cx<T> us[CS][4][9];      // U_mu(x) (link kinds)
  __shared__ T hs[CS][72];            // H(x) (site kind)
  const int wg = xcd_remap(blockIdx.x, gridDim.x);
  const int B = wg / 6, kind = wg - 6 * (wg / 6);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int n = 2 * Nv;
  const int nsites = kind < 2 ? g.bs : g.bs / g.b[kind - 2];
  int bc[4];
  block_coords(g, B, bc);
  acc_t acc[NG][2];
#pragma unroll
  for (int q = 0; q < NG; ++q) acc[q][0] = acc[q][1] = acc_t{0, 0, 0, 0};

  for (int x0 = 0; x0 < nsites; x0 += CS) {
    // stage Q(x), and H(x) or U(x), of the CS sites (zero past the list and past Nv)
    for (int e = t; e < CS * 12 * 32; e += 256) {
      const int xs = e / 384, r = e - xs * 384, c = r >> 5, i = r & 31;
      cx<T> v = mk<T>(0, 0);
      if (x0 + xs < nsites && i < Nv) {
        const int sx = kind < 2 ? x0 + xs : face_slot(g, kind - 2, x0 + xs);
        const cx<RQ> q = Q[(long)i * qstride + fidx(g, B, sx, 12) + (long)c * TILE];
        v = mk<T>((T)q.re, (T)q.im);
      }
      qs[xs][c][i] = v;
    }
    if (kind == 0) {
      for (int e = t; e < CS * 72; e += 256) {
        const int xs = e / 72, k = e - xs * 72;
        hs[xs][k] = x0 + xs < nsites ? (T)H[fidx(g, B, x0 + xs, 72) + (long)k * TILE] : T(0);
      }
    } else {
      for (int e = t; e < CS * 36; e += 256) {
        const int xs = e / 36, k = e - xs * 36;
        cx<T> v = mk<T>(0, 0);
        if (x0 + xs < nsites) {
          const int sx = kind < 2 ? x0 + xs : face_slot(g, kind - 2, x0 + xs);
          const cx<double> ud = U[fidx(g, B, sx, 36) + (long)k * TILE];
          v = mk<T>((T)ud.re, (T)ud.im);
        }
        us[xs][k / 9][k % 9] = v;
      }
    }
    __syncthreads();
    // right factors: one thread per (site, column)
    for (int it = t; it < CS * NC; it += 256) {
      const int xs = it / NC, col = it - xs * NC;
      cx<T> y[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) y[c] = mk<T>(0, 0);
      if (x0 + xs < nsites && col < n) {
        const int hb = col >= Nv ? 1 : 0, j = col - hb * Nv;
        if (kind == 0) {
          cx<T> psi[6], hy[6];
#pragma unroll
          for (int c = 0; c < 6; ++c) psi[c] = qs[xs][6 * hb + c][j];
          herm_mv(&hs[xs][36 * hb], 1, psi, hy);
          if (dtw != 0) {
            // the parity rest of the twist, i d(x) Gamma5 with d = -+ dtw on
            // even / odd sites (Gamma5 = -1 on chirality 0, +1 on chirality 1)
            const T d = (T)((x0 + xs >= g.half) == (hb == 1) ? dtw : -dtw);
#pragma unroll
            for (int c = 0; c < 6; ++c) hy[c] += mk<T>(-d * psi[c].im, d * psi[c].re);
          }
#pragma unroll
          for (int c = 0; c < 6; ++c) {
            y[c] = hb == 0 ? hy[c] : mk<T>(0, 0);
            y[6 + c] = hb == 0 ? mk<T>(0, 0) : hy[c];
          }
        } else {
          const int sx = kind < 2 ? x0 + xs : face_slot(g, kind - 2, x0 + xs);
          SiteNbr me;
          for (int d = 0; d < 4; ++d) me.bc[d] = bc[d];
          slot_local(g, sx, me.l);
          // every direction loads (from x itself when its link is not taken), so
          // that all gathers are in flight together
          bool take[4];
          long off[4];
#pragma unroll
          for (int mu = 0; mu < 4; ++mu) {
            take[mu] = mu < g.ndir && (kind == 1 ? me.l[mu] + 1 < g.b[mu] : mu == kind - 2);
            int By = B, sy = sx;
            if (take[mu]) nbr_of(g, me, mu, +1, By, sy);
            off[mu] = (long)j * qstride + fidx(g, By, sy, 12) + (long)(6 * hb) * TILE;
          }
          cx<RQ> pv[4][6];
#pragma unroll
          for (int mu = 0; mu < 4; ++mu)
#pragma unroll
            for (int c = 0; c < 6; ++c) pv[mu][c] = Q[off[mu] + (long)c * TILE];
          if (take[0]) half_hop<0>(hb, pv[0], us[xs][0], y);
          if (take[1]) half_hop<1>(hb, pv[1], us[xs][1], y);
          if (take[2]) half_hop<2>(hb, pv[2], us[xs][2], y);
          if (take[3]) half_hop<3>(hb, pv[3], us[xs][3], y);
        }
      }
#pragma unroll
      for (int c = 0; c < 12; ++c) ys[xs][c][col] = y[c];
    }
    __syncthreads();
    {
      const int a = w >> 1, i0 = 16 * (w & 1), r16 = lane & 15, kq = lane >> 4;
#pragma unroll
      for (int xs = 0; xs < CS; ++xs)
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          const int kl = 4 * s + kq, c = 6 * a + (kl >> 1), p = kl & 1;
          const cx<T> qv = qs[xs][c][i0 + r16];
          const T av = p ? qv.im : qv.re;
#pragma unroll
          for (int q = 0; q < NG; ++q) {
            const cx<T> yv = ys[xs][c][16 * q + r16];
            const T bre = p ? yv.im : yv.re;
            const T bim = p ? -yv.re : yv.im;
            acc[q][0] = MF::step(av, bre, acc[q][0]);
            acc[q][1] = MF::step(av, bim, acc[q][1]);
          }
        }
    }
    __syncthreads();
  }
  const long site = f2c[B];
  const long nn = (long)n * n;
  cx<double>* out = kind == 1 ? Xs + site * nn : Dc + (site * 5 + (kind == 0 ? 0 : kind - 1)) * nn;
  const int a = w >> 1, i0 = 16 * (w & 1);
#pragma unroll
  for (int q = 0; q < NG; ++q) {
    const int col = 16 * q + (lane & 15);
    if (col >= n) continue;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = i0 + MF::row(lane, e);
      if (i < Nv) out[(long)col * n + a * Nv + i] = mk<double>(acc[q][0][e], acc[q][1][e]);
    }
  }
}
template <class RQ>
void launch_assemble_fine(const Geom& g, int Nv, const cx<double>* U, const double* H, double dtw, const cx<RQ>* Q,
                          long qstride, const int* f2c, cx<double>* Dc, cx<double>* Xs, hipStream_t st) {
  if (Nv < 1 || Nv > 32) throw Error(INVALID_ARG, "assembly: nvec must be in [1, 32]");
  // The Galerkin products are formed and summed in FP64 on the FP64 matrix
  // cores for both storage formats of the test vectors (FP32 vectors are
  // widened as they are staged).  Sites per stage: LDS of two workgroups per CU.
  using T = double;
  constexpr int CS = 4, CS4 = 3;
  const dim3 grid(6 * g.nblocks), blk(256);
  switch ((2 * Nv + 15) / 16) {
    case 1: hipLaunchKernelGGL((k_assemble_fine<RQ, T, CS, 1>), grid, blk, 0, st, g, Nv, U, H, dtw, Q, qstride, f2c, Dc, Xs); break;
    case 2: hipLaunchKernelGGL((k_assemble_fine<RQ, T, CS, 2>), grid, blk, 0, st, g, Nv, U, H, dtw, Q, qstride, f2c, Dc, Xs); break;
    case 3: hipLaunchKernelGGL((k_assemble_fine<RQ, T, CS, 3>), grid, blk, 0, st, g, Nv, U, H, dtw, Q, qstride, f2c, Dc, Xs); break;
    default: hipLaunchKernelGGL((k_assemble_fine<RQ, T, CS4, 4>), grid, blk, 0, st, g, Nv, U, H, dtw, Q, qstride, f2c, Dc, Xs); break;
  }
}
template void launch_assemble_fine<double>(const Geom&, int, const cx<double>*, const double*, double, const cx<double>*,
                                           long, const int*, cx<double>*, cx<double>*, hipStream_t);
template void launch_assemble_fine<float>(const Geom&, int, const cx<double>*, const double*, double, const cx<float>*,
                                          long, const int*, cx<double>*, cx<double>*, hipStream_t);

// ---------------------------------------------------------------------------
// precision copies of operator data
template <class S>
__global__ void k_cvt_cx(long n, const cx<double>* __restrict__ in, typename store_traits<S>::elem* __restrict__ out) {
  long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = st_cvt<S, double>(in[i]);
}
template <class S>
void launch_cvt_cx(long n, const cx<double>* in, void* out, hipStream_t st) {
  hipLaunchKernelGGL(k_cvt_cx<S>, dim3((n + 255) / 256), dim3(256), 0, st, n, in,
                     (typename store_traits<S>::elem*)out);
}
template void launch_cvt_cx<double>(long, const cx<double>*, void*, hipStream_t);
template void launch_cvt_cx<float>(long, const cx<double>*, void*, hipStream_t);
template void launch_cvt_cx<f16>(long, const cx<double>*, void*, hipStream_t);
template void launch_cvt_cx<bf16>(long, const cx<double>*, void*, hipStream_t);

// FP64 operator fields -> copies in 16-byte chunks: nt tiles of 8 sites, per site
// 36 complex link entries in 16 bits (a thread an entry) or 72 reals in FP32 (a
// thread a chunk; us at 48x24x24x24: a thread a chunk of links 100, an entry 85;
// a chunk of reals 94, a real 117).
template <class S>
__global__ void k_chunk_links(long nt, const cx<double>* __restrict__ in,
                              typename store_traits<S>::elem* __restrict__ out) {
  const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= nt * 36 * TILE) return;
  const int lane = (int)(gid % TILE), k = (int)(gid / TILE % 36);
  const long tile = gid / (36 * TILE);
  out[((tile * LC + (k >> 2)) * TILE + lane) * 4 + (k & 3)] = st_cvt<S, double>(in[gid]);
}
template <class S>
void launch_chunk_links(long nt, const cx<double>* in, void* out, hipStream_t st) {
  hipLaunchKernelGGL(k_chunk_links<S>, dim3((unsigned)((nt * 36 * TILE + 255) / 256)), dim3(256), 0, st, nt, in,
                     (typename store_traits<S>::elem*)out);
}
template void launch_chunk_links<f16>(long, const cx<double>*, void*, hipStream_t);
template void launch_chunk_links<bf16>(long, const cx<double>*, void*, hipStream_t);

__global__ void __launch_bounds__(256) k_chunk_real(long nt, const double* __restrict__ in, float4* __restrict__ out) {
  const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= nt * HC * TILE) return;
  const double* p = in + (gid / TILE) * 4 * TILE + gid % TILE;
  out[gid] = float4{(float)p[0], (float)p[TILE], (float)p[2 * TILE], (float)p[3 * TILE]};
}
void launch_chunk_real(long nt, const double* in, float* out, hipStream_t st) {
  hipLaunchKernelGGL(k_chunk_real, dim3((unsigned)((nt * HC * TILE + 255) / 256)), dim3(256), 0, st, nt, in,
                     (float4*)out);
}

// T^{-1} = (H + i tw) M on chirality 0, (H - i tw) M on chirality 1 of every odd
// site, from the FP64 H and M.  One thread per (odd site, chirality), as in
// k_odd_inverse: the packed M stays in registers, H is read a row at a time, and
// every row is stored in whole chunks (48x24x24x24: 117 us, 4.9 TB/s; a thread per
// row reading both 371 us).
__global__ void __launch_bounds__(128) k_chunk_tinv(Geom g, const double* __restrict__ H,
                                                    const double* __restrict__ M, double tw,
                                                    float4* __restrict__ out) {
  const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = (int)(gid & 7), c = (int)(gid >> 3) & 1;
  const long tile = gid >> 4;  // tile of odd sites
  if (tile >= (long)g.nblocks * (g.half / TILE)) return;
  const int B = (int)(tile / (g.half / TILE)), io = (int)(tile % (g.half / TILE)) * TILE + lane;
  const double* hp = H + fidx(g, B, g.half + io, 72) + 36L * c * TILE;
  const double* mp = M + oidx(g, B, io, 72) + 36L * c * TILE;
  double m[36];
#pragma unroll
  for (int k = 0; k < 36; ++k) m[k] = mp[k * TILE];
  auto hget = [hp](int i, int j) {
    if (i == j) return mk(hp[i * TILE], 0.0);
    return i < j ? mk(hp[pk(i, j) * TILE], hp[(pk(i, j) + 1) * TILE])
                 : mk(hp[pk(j, i) * TILE], -hp[(pk(j, i) + 1) * TILE]);
  };
  float4* o = out + (tile * TC + 18 * c) * TILE + lane;
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    cx<double> a[6], row[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) a[k] = hget(i, k);
    a[i].im += c == 0 ? tw : -tw;
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      row[j] = mk(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < 6; ++k) cmac(row[j], a[k], pget(m, k, j));
    }
#pragma unroll
    for (int q = 0; q < 3; ++q)
      o[(3 * i + q) * TILE] =
          float4{(float)row[2 * q].re, (float)row[2 * q].im, (float)row[2 * q + 1].re, (float)row[2 * q + 1].im};
    __builtin_amdgcn_sched_barrier(0);
  }
}
void launch_chunk_tinv(const Geom& g, const double* H, const double* M, double tw, float* out, hipStream_t st) {
  const long n = 2 * (long)g.nblocks * g.half;
  hipLaunchKernelGGL(k_chunk_tinv, dim3((unsigned)((n + 127) / 128)), dim3(128), 0, st, g, H, M, tw, (float4*)out);
}

// ---------------------------------------------------------------------------
// Block orthonormalisation per aggregate half (Sec. 1 aggregation): the
// aggregate's rows of v_1..v_Nv are replaced by Q with V = Q R, R upper
// triangular with a real positive diagonal; that factor is unique, so it is the
// one Gram-Schmidt in the order v_1..v_Nv produces.  It is computed as a
// Cholesky QR in FP64: G = V^H V on the matrix cores, G = R^H R in LDS, then
// Q = V R^{-1} on the matrix cores.  The loss of orthogonality of one pass
// grows like eps64 cond(V)^2: an FP64 output always takes a second pass on Q,
// an FP32 output when the aggregate's smallest pivot ratio R_kk^2 / |v_k|^2 is
// below 1e-6.  A pivot ratio at or below 1e-14 (|R_kk| <= 1e-7 |v_k|, where
// the FP64 Gram matrix no longer resolves the column: linearly dependent test
// vectors) sets *fail.
//
// One workgroup (4 wavefronts) per (block, half); rows r of the aggregate are
// (tile of 8 slots, component of the half, slot in the tile), so 8 consecutive
// rows are contiguous in the block layout.  Nv <= 32 (two 16-wide tiles).
namespace {
constexpr int QR_NT = 256;

__device__ __forceinline__ long qr_row_addr(const Geom& g, int B, int h, int r) {
  const int tau = r / 48, rem = r - 48 * tau, c = rem >> 3, sig = rem & 7;
  return ((long)B * (g.bs / TILE) + tau) * 12 * TILE + (long)(6 * h + c) * TILE + sig;
}

template <class T>
__device__ __forceinline__ cx<double> qr_ld(const cx<T>* p, long stride, int j, int Nv, long a) {
  if (j >= Nv) return mk<double>(0, 0);
  cx<T> v = p[(long)j * stride + a];
  return mk<double>((double)v.re, (double)v.im);
}

// one Cholesky QR pass: src (rows of this aggregate) -> dst; Gr/Gi/Xr/Xi/d0 in LDS
template <class TS, class TD>
__device__ __forceinline__ void cholqr_pass(const Geom& g, int B, int h, int Nv, const cx<TS>* src, long sstride, cx<TD>* dst,
                            long dstride, double (*Gr)[33], double (*Gi)[33], double (*Xr)[33], double (*Xi)[33],
                            double* d0, int* fail, double* ratio) {
  using MF = mfma_k4<double>;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int rows = 6 * g.bs;
  const int NT = Nv > 16 ? 2 : 1;
  const int j0 = lane & 15, kq = lane >> 4, p = kq & 1;
  // ---- G = V^H V: wavefront w sums the complex row pairs ks = w, w+4, ...
  MF::acc a00r = {0, 0, 0, 0}, a00i = {0, 0, 0, 0}, a01r = {0, 0, 0, 0}, a01i = {0, 0, 0, 0}, a11r = {0, 0, 0, 0},
          a11i = {0, 0, 0, 0};
#pragma unroll 4
  for (int ks = w; ks < rows / 2; ks += 4) {
    const long a = qr_row_addr(g, B, h, 2 * ks + (kq >> 1));
    const cx<double> v0 = qr_ld(src, sstride, j0, Nv, a);
    const double x0 = p ? v0.im : v0.re, y0 = p ? -v0.re : v0.im;
    a00r = MF::step(x0, x0, a00r);
    a00i = MF::step(x0, y0, a00i);
    if (NT == 2) {
      const cx<double> v1 = qr_ld(src, sstride, 16 + j0, Nv, a);
      const double x1 = p ? v1.im : v1.re, y1 = p ? -v1.re : v1.im;
      a01r = MF::step(x0, x1, a01r);
      a01i = MF::step(x0, y1, a01i);
      a11r = MF::step(x1, x1, a11r);
      a11i = MF::step(x1, y1, a11i);
    }
  }
  // deterministic sum over the 4 wavefronts, in wavefront order
  for (int v = 0; v < 4; ++v) {
    if (w == v) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = MF::row(lane, e), c = j0;
        Gr[r][c] = (v ? Gr[r][c] : 0.0) + a00r[e];
        Gi[r][c] = (v ? Gi[r][c] : 0.0) + a00i[e];
        if (NT == 2) {
          Gr[r][16 + c] = (v ? Gr[r][16 + c] : 0.0) + a01r[e];
          Gi[r][16 + c] = (v ? Gi[r][16 + c] : 0.0) + a01i[e];
          Gr[16 + r][16 + c] = (v ? Gr[16 + r][16 + c] : 0.0) + a11r[e];
          Gi[16 + r][16 + c] = (v ? Gi[16 + r][16 + c] : 0.0) + a11i[e];
        }
      }
    }
    __syncthreads();
  }
  if (t < Nv) d0[t] = Gr[t][t];
  __syncthreads();
  // ---- G = R^H R in place on the upper triangle (R[k][k] real)
  double rmin = 1.0;  // smallest pivot ratio (thread 0)
  for (int k = 0; k < Nv; ++k) {
    const double dk = Gr[k][k];
    const double rkk = dk > 0 ? sqrt(dk) : 0.0, rinv = rkk > 0 ? 1.0 / rkk : 0.0;
    __syncthreads();
    if (t == 0) {
      const double rk = d0[k] > 0 ? dk / d0[k] : 0.0;
      rmin = rk < rmin ? rk : rmin;
      if (fail && !(rk > 1e-14)) atomicOr(fail, 1);
      Gr[k][k] = rkk;
      Gi[k][k] = 0.0;
    } else if (t > k && t < Nv) {
      Gr[k][t] *= rinv;
      Gi[k][t] *= rinv;
    }
    __syncthreads();
    for (int q = t; q < 32 * 32; q += QR_NT) {
      const int j = q >> 5, l = q & 31;
      if (j > k && l >= j && l < Nv) {
        // G[j][l] -= conj(R[k][j]) R[k][l]
        const double ar = Gr[k][j], ai = Gi[k][j], br = Gr[k][l], bi = Gi[k][l];
        Gr[j][l] -= ar * br + ai * bi;
        Gi[j][l] -= ar * bi - ai * br;
      }
    }
    __syncthreads();
  }
  if (t == 0) *ratio = rmin;
  // ---- X = R^{-1} (upper), one thread per column; zero elsewhere (padding)
  for (int q = t; q < 32 * 32; q += QR_NT) {
    Xr[q >> 5][q & 31] = 0.0;
    Xi[q >> 5][q & 31] = 0.0;
  }
  __syncthreads();
  if (t < Nv) {
    const int i = t;
    Xr[i][i] = Gr[i][i] > 0 ? 1.0 / Gr[i][i] : 0.0;
    for (int j = i - 1; j >= 0; --j) {
      double sr = 0, si = 0;
      for (int m = j + 1; m <= i; ++m) {
        const double ar = Gr[j][m], ai = Gi[j][m], xr = Xr[m][i], xi = Xi[m][i];
        sr += ar * xr - ai * xi;
        si += ar * xi + ai * xr;
      }
      const double ri = Gr[j][j] > 0 ? 1.0 / Gr[j][j] : 0.0;
      Xr[j][i] = -sr * ri;
      Xi[j][i] = -si * ri;
    }
  }
  __syncthreads();
  // ---- Q = V X: wavefront w takes row tiles w, w+4, ...; contraction over (j, re/im)
  const int nks = (Nv + 1) / 2;
  for (int rt = w; rt < rows / 16; rt += 4) {
    const long a = qr_row_addr(g, B, h, 16 * rt + j0);
    MF::acc q0r = {0, 0, 0, 0}, q0i = {0, 0, 0, 0}, q1r = {0, 0, 0, 0}, q1i = {0, 0, 0, 0};
    for (int ks = 0; ks < nks; ++ks) {
      const int j = 2 * ks + (kq >> 1);
      const cx<double> v = qr_ld(src, sstride, j, Nv, a);
      const double av = p ? v.im : v.re;
      const int jj = j < 32 ? j : 31;
      double xr = Xr[jj][j0], xi = Xi[jj][j0];
      q0r = MF::step(av, p ? -xi : xr, q0r);
      q0i = MF::step(av, p ? xr : xi, q0i);
      if (NT == 2) {
        xr = Xr[jj][16 + j0];
        xi = Xi[jj][16 + j0];
        q1r = MF::step(av, p ? -xi : xr, q1r);
        q1i = MF::step(av, p ? xr : xi, q1i);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const long ar = qr_row_addr(g, B, h, 16 * rt + MF::row(lane, e));
      if (j0 < Nv) dst[(long)j0 * dstride + ar] = mk<TD>((TD)q0r[e], (TD)q0i[e]);
      if (NT == 2 && 16 + j0 < Nv) dst[(long)(16 + j0) * dstride + ar] = mk<TD>((TD)q1r[e], (TD)q1i[e]);
    }
  }
  __syncthreads();
}
}  // namespace

template <class RI, class RO>
__global__ void __launch_bounds__(QR_NT) __attribute__((amdgpu_waves_per_eu(3, 8))) k_qr_fine(Geom g, int Nv, const cx<RI>* V, long vstride, RO* Qout_raw,
                                                   long qstride, int* __restrict__ fail) {
  __shared__ double Gr[32][33], Gi[32][33], Xr[32][33], Xi[32][33], d0[32], ratio;
  cx<RO>* Q = reinterpret_cast<cx<RO>*>(Qout_raw);
  const int B = blockIdx.x >> 1, h = blockIdx.x & 1;
  static_assert(std::is_same<RI, RO>::value, "both passes share one body");
  // pass 0 on V; pass 1 on Q for an FP64 output or an ill-conditioned aggregate
  // (ratio is an LDS value after a barrier: uniform over the workgroup)
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    cholqr_pass<RI, RO>(g, B, h, Nv, pass == 0 ? V : reinterpret_cast<const cx<RI>*>(Q),
                        pass == 0 ? vstride : qstride, Q, qstride, Gr, Gi, Xr, Xi, d0, pass == 0 ? fail : nullptr,
                        &ratio);
    if (!(sizeof(RO) == 8 || ratio < 1e-6)) break;
  }
}
template <class RI, class RO>
void launch_qr_fine(const Geom& g, int Nv, const cx<RI>* V, long vstride, cx<RO>* Q, long qstride, int* fail,
                    hipStream_t st) {
  if (Nv < 1 || Nv > 32 || g.bs % TILE) throw Error(INVALID_ARG, "block orthonormalisation needs 1 <= Nv <= 32");
  hipLaunchKernelGGL((k_qr_fine<RI, RO>), dim3(2 * g.nblocks), dim3(QR_NT), 0, st, g, Nv, V, vstride, (RO*)Q, qstride,
                     fail);
}
template void launch_qr_fine<double, double>(const Geom&, int, const cx<double>*, long, cx<double>*, long, int*,
                                             hipStream_t);
template void launch_qr_fine<float, float>(const Geom&, int, const cx<float>*, long, cx<float>*, long, int*,
                                           hipStream_t);

}  // namespace ddamg
