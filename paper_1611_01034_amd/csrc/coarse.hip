// Coarse-level kernels: the coarse operator stencil
//   (D_c y)(c) = S(c) y(c) + i tw Gamma5 y(c)
//               + sum_mu [ F_mu(c) y(c+mu) + Gamma5 F_mu(c-mu)^dag Gamma5 y(c-mu) ]
// (paper Sec. 1: D_c = P^dag D_W P, D_c^dag = Gamma5,c D_c Gamma5,c and
// D_c(mu) = D_c + i mu Gamma5,c), its SAP smoother, restriction / prolongation
// to the next level, block orthonormalisation, Galerkin assembly of the next
// coarse operator, and the odd-even reduced system of the coarsest level
// (Sec. 3: odd-even on the coarsest level).
//
// Storage: vectors [site][n] (n = 2 Nv of the level above, Gamma5,c =
// diag(-1 x n/2, +1 x n/2)); operator [site][5][n][n], block 0 = S without the
// twist, block 1+mu = F_mu, each block column-major (element (k,l) at l*n+k).
// Sites are numbered even parity first, so the even half of a vector is a
// prefix.  One wavefront handles one site; lane k computes row k (n <= 64).
#include "kernels.hpp"

namespace ddamg {

__device__ __forceinline__ double g5(int k, int n) { return k < (n >> 1) ? -1.0 : 1.0; }

template <class R, class S>
__device__ __forceinline__ cx<R> Dld(const typename store_traits<S>::elem* D, long idx) {
  return ld<R, S>(D, idx);
}

// stage y at the site (slot 0) and its 8 neighbours (slots 1..8) in LDS
template <class R>
__device__ __forceinline__ void stage9(cx<R> (*ys)[64], const CGeom& cg, int site, bool valid, const cx<R>* in,
                                       int lane) {
  if (valid && lane < cg.n) {
    ys[0][lane] = in[(long)site * cg.n + lane];
#pragma unroll
    for (int j = 0; j < 8; ++j) ys[1 + j][lane] = in[(long)cg.nbr[site * 8 + j] * cg.n + lane];
  }
}

template <class R, class S>
__device__ __forceinline__ cx<R> self_row(const CGeom& cg, const typename store_traits<S>::elem* D, int site, int k,
                                          R tw, const cx<R>* y) {
  const int n = cg.n;
  long base = (long)site * 5 * n * n;
  cx<R> acc = mk<R>(0, 0);
  for (int l = 0; l < n; ++l) cmac(acc, Dld<R, S>(D, base + (long)l * n + k), y[l]);
  acc += (R)(tw * g5(k, n)) * times_i(y[k]);
  return acc;
}

template <class R, class S>
__device__ __forceinline__ cx<R> hop_row(const CGeom& cg, const typename store_traits<S>::elem* D, int site, int k,
                                         cx<R> (*ys)[64]) {
  const int n = cg.n;
  const long nn = (long)n * n;
  cx<R> acc = mk<R>(0, 0);
#pragma unroll 1
  for (int mu = 0; mu < 4; ++mu) {
    long bf = ((long)site * 5 + 1 + mu) * nn;
    const cx<R>* yf = ys[1 + mu];
    for (int l = 0; l < n; ++l) cmac(acc, Dld<R, S>(D, bf + (long)l * n + k), yf[l]);
    int cb = cg.nbr[site * 8 + 4 + mu];
    long bb = ((long)cb * 5 + 1 + mu) * nn + (long)k * n;
    const cx<R>* yb = ys[5 + mu];
    cx<R> t = mk<R>(0, 0);
    const int h = n >> 1;
    for (int l = 0; l < h; ++l) cjmac(t, Dld<R, S>(D, bb + l), yb[l]);
    cx<R> t2 = mk<R>(0, 0);
    for (int l = h; l < n; ++l) cjmac(t2, Dld<R, S>(D, bb + l), yb[l]);
    // g_k * (g_l sums): lower half g_l = -1, upper half +1
    cx<R> tb = t2 - t;
    if (k < h) acc -= tb;
    else acc += tb;
  }
  return acc;
}

// ---------------------------------------------------------------------------
// One site per workgroup of eight wavefronts, for grids whose sites do not fill
// the card at one wavefront each: wavefront w takes one of the eight hops (and
// an eighth of the self block's columns), so that the site's blocks are loaded
// together instead of one after the other.  Lanes hold rows; with n <= 32 the
// lanes left over split the inner index P ways.  Sums are in R as in the
// one-wavefront form, the 8 P partial sums of a row added in fixed order.
namespace {
constexpr int SITE_W = 8;
constexpr int SITE_T = 64 * SITE_W;
// inner-index parts per wavefront
__device__ __forceinline__ int site_parts(int n) { return n > 32 ? 1 : n > 16 ? 2 : n > 8 ? 4 : 8; }

// sum over l = l0 + part, l0 + part + P, ... < l1 of D[l * n + k] y[l]
template <class R, class S>
__device__ __forceinline__ cx<R> col_sum(const typename store_traits<S>::elem* D, int n, int k, int l0, int l1, int P,
                                         const cx<R>* y) {
  constexpr int U = sizeof(R) == 8 ? 8 : 16;  // entries in flight
  cx<R> acc = mk<R>(0, 0);
  for (int l = l0; l < l1; l += U * P) {
    cx<R> d[U];
#pragma unroll
    for (int q = 0; q < U; ++q) d[q] = ld<R, S>(D, (long)min(l + q * P, l1 - 1) * n + k);
#pragma unroll
    for (int q = 0; q < U; ++q)
      if (l + q * P < l1) cmac(acc, d[q], y[l + q * P]);
  }
  return acc;
}
// sum over the l of this part of conj(D[k * n + l]) y[l]: a lane reads its row
// VE entries (16 bytes) at a time where n allows
template <class R, class S>
__device__ __forceinline__ cx<R> row_sum(const typename store_traits<S>::elem* D, int n, int k, int part, int P,
                                         const cx<R>* y) {
  using E = typename store_traits<S>::elem;
  constexpr int VE = 16 / sizeof(E), U = sizeof(R) == 8 ? 8 : 4;
  struct alignas(16) V {
    E e[VE];
  };
  cx<R> acc = mk<R>(0, 0);
  if (n % VE == 0) {
    const V* p = reinterpret_cast<const V*>(D + (long)k * n);
    const int nv = n / VE;
    for (int c = part; c < nv; c += U * P) {
      V v[U];
#pragma unroll
      for (int q = 0; q < U; ++q) v[q] = p[min(c + q * P, nv - 1)];
#pragma unroll
      for (int q = 0; q < U; ++q)
        if (c + q * P < nv) {
#pragma unroll
          for (int e = 0; e < VE; ++e) cjmac(acc, ld<R, S>(v[q].e, e), y[(c + q * P) * VE + e]);
        }
    }
  } else {
    for (int l = part; l < n; l += P) cjmac(acc, ld<R, S>(D, (long)k * n + l), y[l]);
  }
  return acc;
}

// partial sums ps[(w P + part) * n + row] of hs * (hops of xh) + S xs at `site`
// (xs null: hops only); ys: 9 * 64 complex of LDS.  Ends with a barrier.
template <class R, class S>
__device__ __forceinline__ void site_partials(const CGeom& cg, const typename store_traits<S>::elem* D, int site,
                                              const cx<R>* xs, const cx<R>* xh, R hs, cx<R>* ys, cx<R>* ps) {
  const int n = cg.n, h = n >> 1, P = site_parts(n), rows = 64 / P;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long nn = (long)n * n;
  const int row = lane & (rows - 1), part = lane / rows, nb = cg.nbr[site * 8 + w];
  // the wavefront's hop input (the backward one with its Gamma5 sign) and an
  // eighth of the self input
  if (lane < n) {
    const cx<R> v = xh[(long)nb * n + lane];
    const R f = w >= 4 && lane < h ? -hs : hs;
    ys[w * 64 + lane] = mk<R>(f * v.re, f * v.im);
  }
  const int l0 = w * n / SITE_W, l1 = (w + 1) * n / SITE_W;
  if (xs && lane >= l0 && lane < l1) ys[8 * 64 + lane] = xs[(long)site * n + lane];
  __syncthreads();
  if (row < n) {
    cx<R> acc;
    if (w < 4) {
      acc = col_sum<R, S>(D + ((long)site * 5 + 1 + w) * nn, n, row, part, n, P, ys + w * 64);
    } else {
      acc = row_sum<R, S>(D + ((long)nb * 5 + 1 + (w - 4)) * nn, n, row, part, P, ys + w * 64);
      if (row < h) acc = -acc;
    }
    if (xs) acc += col_sum<R, S>(D + (long)site * 5 * nn, n, row, l0 + part, l1, P, ys + 8 * 64);
    ps[(w * P + part) * n + row] = acc;
  }
  __syncthreads();
}
template <class R>
__device__ __forceinline__ cx<R> site_sum(const CGeom& cg, const cx<R>* ps, int k) {
  const int q = SITE_W * site_parts(cg.n);
  cx<R> v = mk<R>(0, 0);
  for (int p = 0; p < q; ++p) v += ps[p * cg.n + k];
  return v;
}
}  // namespace

// out = D y, or b - D y
template <class R, class S>
__global__ void __launch_bounds__(SITE_T) k_coarse_apply_site(CGeom cg,
                                                              const typename store_traits<S>::elem* __restrict__ D, R tw,
                                                              const cx<R>* __restrict__ in, const cx<R>* __restrict__ b,
                                                              cx<R>* __restrict__ out) {
  __shared__ cx<R> ys[9 * 64], ps[SITE_T];
  // each XCD takes a contiguous range of sites in lexicographic order: a
  // forward block is still in its L2 when the neighbours' backward hops read it
  const int site = cg.lexord[xcd_remap(blockIdx.x, gridDim.x)], k = threadIdx.x, n = cg.n;
  site_partials<R, S>(cg, D, site, in, in, R(1), ys, ps);
  if (k >= n) return;
  const long o = (long)site * n + k;
  const cx<R> acc = site_sum(cg, ps, k) + (R)(tw * g5(k, n)) * times_i(in[o]);
  out[o] = b ? b[o] - acc : acc;
}

// even sites: mode 0: out = (S + i tw G5) v - hop(t);  mode 1: out = v - hop(t)
template <class R, class S>
__global__ void __launch_bounds__(SITE_T) k_coarse_schur_even_site(CGeom cg,
                                                                   const typename store_traits<S>::elem* __restrict__ D,
                                                                   R tw, const cx<R>* __restrict__ v,
                                                                   const cx<R>* __restrict__ tv, cx<R>* __restrict__ out,
                                                                   int mode) {
  __shared__ cx<R> ys[9 * 64], ps[SITE_T];
  const int site = blockIdx.x, k = threadIdx.x, n = cg.n;
  site_partials<R, S>(cg, D, site, mode == 0 ? v : nullptr, tv, R(-1), ys, ps);
  if (k >= n) return;
  const long o = (long)site * n + k;
  const cx<R> acc = site_sum(cg, ps, k), x = v[o];
  out[o] = mode == 0 ? acc + (R)(tw * g5(k, n)) * times_i(x) : x + acc;
}

// odd sites: out = M (base - hop(in)) if base, else out = M hop(in)
template <class R, class S>
__global__ void __launch_bounds__(SITE_T) k_coarse_hop_inv_odd_site(CGeom cg,
                                                                    const typename store_traits<S>::elem* __restrict__ D,
                                                                    const cx<R>* __restrict__ Minv,
                                                                    const cx<R>* __restrict__ in,
                                                                    const cx<R>* __restrict__ base,
                                                                    cx<R>* __restrict__ out) {
  __shared__ cx<R> ys[9 * 64], ps[SITE_T];
  const int n = cg.n, io = blockIdx.x, site = cg.neven + io, t = threadIdx.x;
  // this thread's entries of the inverse (row, l = q, q + 8 P, ...: at most 8),
  // loaded before the hops
  const int P = site_parts(n), rows = 64 / P, Q = SITE_W * P, row = t & (rows - 1), q = t / rows;
  const cx<R>* M = Minv + (long)io * n * n;
  cx<R> m[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) m[j] = M[(long)min(q + j * Q, n - 1) * n + min(row, n - 1)];
  site_partials<R, S>(cg, D, site, nullptr, in, R(1), ys, ps);
  if (t < n) {
    cx<R> u = site_sum(cg, ps, t);
    if (base) u = base[(long)site * n + t] - u;
    ys[t] = u;
  }
  __syncthreads();
  cx<R> acc = mk<R>(0, 0);
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (q + j * Q < n) cmac(acc, m[j], ys[q + j * Q]);
  if (row < n) ps[q * n + row] = acc;
  __syncthreads();
  if (t < n) {
    cx<R> o = mk<R>(0, 0);
    for (int p = 0; p < Q; ++p) o += ps[p * n + t];
    out[(long)site * n + t] = o;
  }
}

// out = D y   (or out = b - D y when b != nullptr)
template <class R, class S>
__global__ void __launch_bounds__(256) k_coarse_apply(CGeom cg, const typename store_traits<S>::elem* __restrict__ D,
                                                      R tw, const cx<R>* __restrict__ in, const cx<R>* __restrict__ b,
                                                      cx<R>* __restrict__ out) {
  __shared__ cx<R> ys[4][9][64];
  int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int site = blockIdx.x * 4 + wv;
  bool valid = site < cg.nsites;
  stage9(ys[wv], cg, site, valid, in, lane);
  __syncthreads();
  if (valid && lane < cg.n) {
    cx<R> acc = self_row<R, S>(cg, D, site, lane, tw, ys[wv][0]) + hop_row<R, S>(cg, D, site, lane, ys[wv]);
    long o = (long)site * cg.n + lane;
    out[o] = b ? b[o] - acc : acc;
  }
}

// Whether a launch over nsites sites (of one parity in the odd-even operator) takes
// one workgroup per site.  From n = 26 on it is as fast or faster on every size
// measured (us, before and now; apply: FP64 n = 48 on 32 sites 31 and 11, on 2048
// 116 and 115, on 8192 620 and 452; FP32 n = 64 on 512 55 and 27; odd-even pair:
// 16-bit n = 52 on 1024 94 and 30).
// Smaller sites give eight wavefronts too little work once the grid fills the
// card (FP32 n = 16: pair on 512 sites 23 and 11, apply on 1024 10.5 and 11.9,
// on 8192 45 and 82).
static inline bool one_site(int nsites, int n) { return n > 24 || nsites <= 512; }
template <class R, class S>
static void coarse_apply(const CGeom& cg, const void* D, double tw, const cx<R>* in, const cx<R>* b, cx<R>* out,
                         hipStream_t st) {
  auto Dp = (const typename store_traits<S>::elem*)D;
  if (one_site(cg.nsites, cg.n))
    hipLaunchKernelGGL((k_coarse_apply_site<R, S>), dim3(cg.nsites), dim3(SITE_T), 0, st, cg, Dp, (R)tw, in, b, out);
  else
    hipLaunchKernelGGL((k_coarse_apply<R, S>), dim3((cg.nsites + 3) / 4), dim3(256), 0, st, cg, Dp, (R)tw, in, b, out);
}
template <class R, class S>
void launch_coarse_apply(const CGeom& cg, const void* D, double tw, const cx<R>* in, cx<R>* out, hipStream_t st) {
  coarse_apply<R, S>(cg, D, tw, in, nullptr, out, st);
}
template <class R, class S>
void launch_coarse_residual(const CGeom& cg, const void* D, double tw, const cx<R>* b, const cx<R>* x, cx<R>* r,
                            hipStream_t st) {
  coarse_apply<R, S>(cg, D, tw, x, b, r, st);
}

// ---------------------------------------------------------------------------
// coarse SAP: one workgroup per block of the colour, one wavefront per block
// site; n_mr MR steps on the Dirichlet block operator D_B.
template <class R, class S>
__global__ void __launch_bounds__(1024) k_coarse_sap(CGeom cg, const typename store_traits<S>::elem* __restrict__ D,
                                                     R tw, int bsz, const int* __restrict__ blk_sites,
                                                     const int* __restrict__ blk_nbr, const cx<R>* __restrict__ r,
                                                     cx<R>* __restrict__ x, int n_mr, int K, long ld) {
  extern __shared__ char smem_raw[];
  cx<R>* rho = reinterpret_cast<cx<R>*>(smem_raw);  // [bsz][64]
  __shared__ double red[3][16];
  const int n = cg.n;
  const long nn = (long)n * n;
  // K fields interleaved: consecutive workgroups take one block for different fields
  const int blk = blockIdx.x / K, rr = blockIdx.x - blk * K;
  r += (long)rr * ld;
  x += (long)rr * ld;
  int j = threadIdx.x >> 6, k = threadIdx.x & 63;
  int site = blk_sites[blk * bsz + j];
  const int* lnb = blk_nbr + ((long)blk * bsz + j) * 8;
  bool act = k < n;
  rho[j * 64 + k] = act ? r[(long)site * n + k] : mk<R>(0, 0);
  cx<R> eps = mk<R>(0, 0);
  const int h = n >> 1;
  for (int it = 0; it < n_mr; ++it) {
    __syncthreads();
    cx<R> q = mk<R>(0, 0);
    if (act) {
      q = self_row<R, S>(cg, D, site, k, tw, rho + j * 64);
      for (int mu = 0; mu < 4; ++mu) {
        int jf = lnb[mu];
        if (jf >= 0) {
          long bf = ((long)site * 5 + 1 + mu) * nn;
          const cx<R>* yf = rho + jf * 64;
          for (int l = 0; l < n; ++l) cmac(q, Dld<R, S>(D, bf + (long)l * n + k), yf[l]);
        }
        int jb = lnb[4 + mu];
        if (jb >= 0) {
          int cb = blk_sites[blk * bsz + jb];
          long bb = ((long)cb * 5 + 1 + mu) * nn + (long)k * n;
          const cx<R>* yb = rho + jb * 64;
          cx<R> t = mk<R>(0, 0), t2 = mk<R>(0, 0);
          for (int l = 0; l < h; ++l) cjmac(t, Dld<R, S>(D, bb + l), yb[l]);
          for (int l = h; l < n; ++l) cjmac(t2, Dld<R, S>(D, bb + l), yb[l]);
          cx<R> tb = t2 - t;
          if (k < h) q -= tb;
          else q += tb;
        }
      }
    }
    cx<R> rk = rho[j * 64 + k];
    double qr_re = (double)q.re * rk.re + (double)q.im * rk.im;
    double qr_im = (double)q.re * rk.im - (double)q.im * rk.re;
    double qq = (double)q.re * q.re + (double)q.im * q.im;
    qr_re = wave_sum_n(qr_re, 64);
    qr_im = wave_sum_n(qr_im, 64);
    qq = wave_sum_n(qq, 64);
    if (k == 0) {
      red[0][j] = qr_re;
      red[1][j] = qr_im;
      red[2][j] = qq;
    }
    __syncthreads();
    double sr = 0, si = 0, sq = 0;
    for (int v = 0; v < bsz; ++v) {
      sr += red[0][v];
      si += red[1][v];
      sq += red[2][v];
    }
    cx<R> alpha = mk<R>(0, 0);
    if (sq > 0) alpha = mk<R>((R)(sr / sq), (R)(si / sq));
    eps += alpha * rk;
    rho[j * 64 + k] = rk - alpha * q;
  }
  if (act) {
    long o = (long)site * n + k;
    x[o] = x[o] + eps;
  }
}

template <class R, class S>
void launch_coarse_sap(const CGeom& cg, const void* D, double tw, int nblk_colour, int bsz, const int* blk_sites,
                       const int* blk_nbr, const cx<R>* r, cx<R>* x, int n_mr, hipStream_t st) {
  launch_coarse_sap_multi<R, S>(cg, D, tw, nblk_colour, bsz, blk_sites, blk_nbr, r, x, n_mr, 1, 0, st);
}
template <class R, class S>
void launch_coarse_sap_multi(const CGeom& cg, const void* D, double tw, int nblk_colour, int bsz, const int* blk_sites,
                             const int* blk_nbr, const cx<R>* r, cx<R>* x, int n_mr, int K, long ld, hipStream_t st) {
  size_t sm = (size_t)bsz * 64 * sizeof(cx<R>);
  hipLaunchKernelGGL((k_coarse_sap<R, S>), dim3(nblk_colour * K), dim3(64 * bsz), sm, st, cg,
                     (const typename store_traits<S>::elem*)D, (R)tw, bsz, blk_sites, blk_nbr, r, x, n_mr, K, ld);
}

// ---------------------------------------------------------------------------
// restriction to the next level: r_c[A][s*Nv+i] = sum_{j in A, k in half s}
// conj(Q_i[site_j][k]) r[site_j][k].  One workgroup (256) per aggregate (and
// column); wavefront w takes the vectors 8w..8w+7 (then +32, ...) over the
// entries of one half after the other (lanes on consecutive entries) and sums its
// 32 values (8 vectors x 2 halves x re/im) with one transposing wavefront sum: no
// LDS, no barriers, the four wavefronts independent.  Bound by instructions: both
// halves at once, each entry selected for one and divided into (site, component),
// took three times as many (32 vectors on 256 aggregates of 768 entries, six
// columns: 99 -> 79 us).
template <class R>
__device__ __forceinline__ void restrict_column(int n, int Nv, int asz, const int* sites, const cx<R>* Q, long qstride,
                                                const cx<R>* r, cx<R>* rc) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int hn = n >> 1, dj = 64 / hn, dk = 64 - dj * hn;
  const int j0 = lane / hn, k0 = lane - j0 * hn;
  for (int i0 = 8 * w; i0 < Nv; i0 += 32) {
    double acc[32];  // [4 ii + 2 h + p]
#pragma unroll
    for (int q = 0; q < 32; ++q) acc[q] = 0.0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      int j = j0, k = k0;
#pragma unroll 2
      while (j < asz) {
        const long idx = (long)sites[j] * n + h * hn + k;
        const cx<R> rv = r[idx];
#pragma unroll
        for (int ii = 0; ii < 8; ++ii) {
          const int iv = i0 + ii < Nv ? i0 + ii : Nv - 1;  // clamped: every load in flight
          const cx<R> qv = Q[(long)iv * qstride + idx];
          acc[4 * ii + 2 * h] += (double)qv.re * rv.re + (double)qv.im * rv.im;
          acc[4 * ii + 2 * h + 1] += (double)qv.re * rv.im - (double)qv.im * rv.re;
        }
        j += dj;
        k += dk;
        if (k >= hn) {
          k -= hn;
          ++j;
        }
      }
    }
    const double v = wave_transpose_sum<32>(acc, lane);  // lane l: total of value l % 32
    if (lane < 32) {
      const int ii = lane >> 2, hh = (lane >> 1) & 1, p = lane & 1;
      if (i0 + ii < Nv) reinterpret_cast<R*>(rc + hh * Nv + i0 + ii)[p] = (R)v;
    }
  }
}
template <class R>
__global__ void __launch_bounds__(256) k_restrict_coarse(int n, int Nv, int asz, const int* __restrict__ agg_sites,
                                                         const cx<R>* __restrict__ Q, long qstride,
                                                         const cx<R>* __restrict__ r, cx<R>* __restrict__ rc) {
  const int A = blockIdx.x;
  restrict_column(n, Nv, asz, agg_sites + A * asz, Q, qstride, r, rc + (long)A * 2 * Nv);
}
template <class R>
void launch_restrict_coarse(int n, int Nv, int nagg, int asz, const int* agg_sites, const cx<R>* Q, long qstride,
                            const cx<R>* r, cx<R>* rc, hipStream_t st) {
  hipLaunchKernelGGL(k_restrict_coarse<R>, dim3(nagg), dim3(256), 0, st, n, Nv, asz, agg_sites, Q, qstride, r, rc);
}

// K columns (stride rld in, cld out): one workgroup per (aggregate, column),
// the K columns of an aggregate in consecutive workgroups of one XCD, so its
// part of Q comes from HBM once and from L2 for the other columns
template <class R>
__global__ void __launch_bounds__(256) k_restrict_coarse_m(int n, int Nv, int asz, const int* __restrict__ agg_sites,
                                                           const cx<R>* __restrict__ Q, long qstride,
                                                           const cx<R>* __restrict__ r, long rld,
                                                           cx<R>* __restrict__ rc, long cld, int K) {
  const int wq = xcd_remap(blockIdx.x, gridDim.x), A = wq / K, col = wq - A * K;
  restrict_column(n, Nv, asz, agg_sites + A * asz, Q, qstride, r + (long)col * rld,
                  rc + (long)col * cld + (long)A * 2 * Nv);
}
template <class R>
void launch_restrict_coarse_m(int n, int Nv, int nagg, int asz, const int* agg_sites, const cx<R>* Q, long qstride,
                              const cx<R>* r, long rld, cx<R>* rc, long cld, int K, hipStream_t st) {
  hipLaunchKernelGGL(k_restrict_coarse_m<R>, dim3(nagg * K), dim3(256), 0, st, n, Nv, asz, agg_sites, Q, qstride, r,
                     rld, rc, cld, K);
}

// K columns: one thread per entry for all columns, in groups of KC whose
// accumulators stay in registers (Q read once per group)
template <class R, int KC>
__global__ void k_prolong_coarse_m(int n, int Nv, int nsites, const int* __restrict__ site_agg,
                                   const cx<R>* __restrict__ Q, long qstride, const cx<R>* __restrict__ ec, long cld,
                                   cx<R>* __restrict__ x, long xld, int K, int accumulate) {
  const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long)nsites * n) return;
  const int site = (int)(gid / n), k = (int)(gid - (long)site * n);
  const int h = k >= (n >> 1) ? 1 : 0;
  const cx<R>* e = ec + (long)site_agg[site] * 2 * Nv + h * Nv;
  for (int k0 = 0; k0 < K; k0 += KC) {
    cx<R> acc[KC];
#pragma unroll
    for (int kk = 0; kk < KC; ++kk)
      acc[kk] = accumulate && k0 + kk < K ? x[(long)(k0 + kk) * xld + gid] : mk<R>(0, 0);
    for (int i = 0; i < Nv; ++i) {
      const cx<R> q = Q[(long)i * qstride + gid];
#pragma unroll
      for (int kk = 0; kk < KC; ++kk)
        if (k0 + kk < K) cmac(acc[kk], q, e[(long)(k0 + kk) * cld + i]);
    }
#pragma unroll
    for (int kk = 0; kk < KC; ++kk)
      if (k0 + kk < K) x[(long)(k0 + kk) * xld + gid] = acc[kk];
  }
}
template <class R>
void launch_prolong_coarse_m(int n, int Nv, int nsites, const int* site_agg, const cx<R>* Q, long qstride,
                             const cx<R>* ec, long cld, cx<R>* x, long xld, int K, int accumulate, hipStream_t st) {
  const long tot = (long)nsites * n;
  const dim3 grid((unsigned)((tot + 255) / 256)), blk(256);
  if (K <= 4)
    hipLaunchKernelGGL((k_prolong_coarse_m<R, 4>), grid, blk, 0, st, n, Nv, nsites, site_agg, Q, qstride, ec, cld, x,
                       xld, K, accumulate);
  else
    hipLaunchKernelGGL((k_prolong_coarse_m<R, 8>), grid, blk, 0, st, n, Nv, nsites, site_agg, Q, qstride, ec, cld, x,
                       xld, K, accumulate);
}

template <class R>
__global__ void k_prolong_coarse(int n, int Nv, int nsites, const int* __restrict__ site_agg,
                                 const cx<R>* __restrict__ Q, long qstride, const cx<R>* __restrict__ ec,
                                 cx<R>* __restrict__ x, int accumulate) {
  long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long)nsites * n) return;
  int site = (int)(gid / n), k = (int)(gid - (long)site * n);
  int h = k >= (n >> 1) ? 1 : 0;
  const cx<R>* e = ec + (long)site_agg[site] * 2 * Nv + h * Nv;
  cx<R> acc = accumulate ? x[gid] : mk<R>(0, 0);
  for (int i = 0; i < Nv; ++i) cmac(acc, Q[(long)i * qstride + gid], e[i]);
  x[gid] = acc;
}
template <class R>
void launch_prolong_coarse(int n, int Nv, int nsites, const int* site_agg, const cx<R>* Q, long qstride,
                           const cx<R>* ec, cx<R>* x, int accumulate, hipStream_t st) {
  long tot = (long)nsites * n;
  hipLaunchKernelGGL(k_prolong_coarse<R>, dim3((tot + 255) / 256), dim3(256), 0, st, n, Nv, nsites, site_agg, Q,
                     qstride, ec, x, accumulate);
}

// ---------------------------------------------------------------------------
// block orthonormalisation on a coarse level (CGS2, FP64), one workgroup per
// (aggregate, half), one thread per row (site j, component c of the half)
template <class RI, class RO>
__global__ void __launch_bounds__(1024) k_qr_coarse(int n, int Nv, int asz, const int* __restrict__ agg_sites,
                                                    const cx<RI>* __restrict__ V, long vstride,
                                                    RO* __restrict__ Qraw, long qstride, int* __restrict__ fail) {
  cx<RO>* Qout = reinterpret_cast<cx<RO>*>(Qraw);
  __shared__ double red[32][16][2];
  __shared__ double dsh[32][2];
  int A = blockIdx.x >> 1, h = blockIdx.x & 1;
  int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int hn = n >> 1, rows = asz * hn;
  const int nw = (rows + 63) >> 6;
  const int nact = min(64, rows - wv * 64);
  bool act = t < rows;
  long idx = 0;
  if (act) {
    int j = t / hn, c = t - j * hn;
    idx = (long)agg_sites[A * asz + j] * n + h * hn + c;
  }
  auto reduce = [&](double a, double b, int slot) {
    a = wave_sum_n(a, nact);
    b = wave_sum_n(b, nact);
    if (lane == 0) {
      red[slot][wv][0] = a;
      red[slot][wv][1] = b;
    }
  };
  for (int i = 0; i < Nv; ++i) {
    cx<double> v = mk(0.0, 0.0);
    if (act) {
      cx<RI> vi = V[(long)i * vstride + idx];
      v = mk<double>(vi.re, vi.im);
    }
    reduce(norm2(v), 0.0, 0);
    __syncthreads();
    double nrm0 = 0;
    for (int w = 0; w < nw; ++w) nrm0 += red[0][w][0];
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
      for (int jj = 0; jj < i; ++jj) {
        double ar = 0, ai = 0;
        if (act) {
          cx<RO> q = Qout[(long)jj * qstride + idx];
          ar = (double)q.re * v.re + (double)q.im * v.im;
          ai = (double)q.re * v.im - (double)q.im * v.re;
        }
        reduce(ar, ai, jj);
      }
      __syncthreads();
      if (t < i) {
        double re = 0, im = 0;
        for (int w = 0; w < nw; ++w) {
          re += red[t][w][0];
          im += red[t][w][1];
        }
        dsh[t][0] = re;
        dsh[t][1] = im;
      }
      __syncthreads();
      if (act)
        for (int jj = 0; jj < i; ++jj) {
          cx<RO> q = Qout[(long)jj * qstride + idx];
          v = v - mk(dsh[jj][0], dsh[jj][1]) * mk<double>(q.re, q.im);
        }
      __syncthreads();
    }
    reduce(norm2(v), 0.0, 0);
    __syncthreads();
    double nrm = 0;
    for (int w = 0; w < nw; ++w) nrm += red[0][w][0];
    __syncthreads();
    if (!(nrm > 1e-24 * nrm0) && t == 0) atomicOr(fail, 1);
    double inv = nrm > 0 ? 1.0 / sqrt(nrm) : 0.0;
    if (act) Qout[(long)i * qstride + idx] = mk<RO>((RO)(inv * v.re), (RO)(inv * v.im));
  }
}
template <class RI, class RO>
void launch_qr_coarse(int n, int Nv, int nagg, int asz, const int* agg_sites, const cx<RI>* V, long vstride,
                      cx<RO>* Q, long qstride, int* fail, hipStream_t st) {
  int rows = asz * (n / 2);
  int threads = ((rows + 63) / 64) * 64;
  hipLaunchKernelGGL((k_qr_coarse<RI, RO>), dim3(2 * nagg), dim3(threads), 0, st, n, Nv, asz, agg_sites, V, vstride,
                     (RO*)Q, qstride, fail);
}

// ---------------------------------------------------------------------------
// Galerkin assembly of the next coarse operator from a coarse level, FP64.
// One workgroup per (aggregate A, kind): kind 0 = self (site blocks + links
// inside A), kind 1+mu = forward block (links across the upper mu face).
// q = Q(c) staged per site, Q(y) staged per piece; W = (operator block) * Q(y)
// per half of the output columns, one thread per (component k, group of 8
// vectors): each operator entry is loaded once (all loads in flight) and used
// for the 8 vectors from LDS.
template <class RQ>
__global__ void __launch_bounds__(256) k_assemble_coarse(CGeom cg, int Nv, int a0, int a1, int a2, int a3,
                                                         const int* __restrict__ agg_sites,
                                                         const cx<double>* __restrict__ D,
                                                         const cx<RQ>* __restrict__ Q, long qstride,
                                                         cx<double>* __restrict__ Dn, cx<double>* __restrict__ Xs) {
  const int n = cg.n, hn = n >> 1, np = 2 * Nv;
  const long nn = (long)n * n;
  const int asz = a0 * a1 * a2 * a3;
  const int ab[4] = {a0, a1, a2, a3};
  extern __shared__ char smem_raw[];
  // q rows padded to n + 1 entries: the output sums read 32 rows at one k
  cx<double>* q = reinterpret_cast<cx<double>*>(smem_raw);  // q[i][k] = Q_i(c)[k] at i (n + 1) + k
  cx<double>* W = q + Nv * (n + 1);                           // W[i][k] for output columns of one half
  cx<double>* qy = W + Nv * n;                                // qy[i][k] = Q_i(y)[k]
  // workgroup = (aggregate, kind, half hc of the output columns)
  const int A = blockIdx.x / 10, kind = (blockIdx.x % 10) >> 1, hc = blockIdx.x & 1;
  int t = threadIdx.x;
  const int nent = np * np, nh = Nv * np;  // entries per column half: e = hc nh + t + 256 m
  cx<double> accS[8], accX[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) accS[m] = accX[m] = mk(0.0, 0.0);
  for (int j = 0; j < asz; ++j) {
    int l[4];
    {
      int r = j;
      l[3] = r % a3;
      r /= a3;
      l[2] = r % a2;
      r /= a2;
      l[1] = r % a1;
      l[0] = r / a1;
    }
    if (kind > 0 && l[kind - 1] != ab[kind - 1] - 1) continue;
    int c = agg_sites[A * asz + j];
    __syncthreads();
    for (int e = t; e < Nv * n; e += 256) {
      int i = e / n, k = e - i * n;
      cx<RQ> v = Q[(long)i * qstride + (long)c * n + k];
      q[i * (n + 1) + k] = mk<double>(v.re, v.im);
    }
    // pieces: piece -1 = site block, piece mu = forward link in direction mu
    for (int piece = -1; piece < 4; ++piece) {
      int y;
      long blk;
      if (piece < 0) {
        if (kind != 0) continue;
        y = c;
        blk = (long)c * 5 * nn;
      } else {
        bool take = (kind == 0) ? (l[piece] + 1 < ab[piece]) : (piece == kind - 1);
        if (!take) continue;
        y = cg.nbr[c * 8 + piece];
        blk = ((long)c * 5 + 1 + piece) * nn;
      }
      bool toX = (kind == 0 && piece >= 0);
      __syncthreads();
      for (int e = t; e < Nv * n; e += 256) {
        int i = e / n, k = e - i * n;
        cx<RQ> v = Q[(long)i * qstride + (long)y * n + k];
        qy[e] = mk<double>(v.re, v.im);
      }
      {
        __syncthreads();
        // W[i][k] = sum_{k2 in half hc} B[k][k2] Q_i(y)[k2]
        const int ng = (Nv + 7) / 8;
        for (int task = t; task < n * ng; task += 256) {
          const int k = task % n, i0 = 8 * (task / n);
          cx<double> acc[8];
#pragma unroll
          for (int ii = 0; ii < 8; ++ii) acc[ii] = mk(0.0, 0.0);
#pragma unroll 4
          for (int k2 = hc * hn; k2 < (hc + 1) * hn; ++k2) {
            const cx<double> d = D[blk + (long)k2 * n + k];
#pragma unroll
            for (int ii = 0; ii < 8; ++ii)
              if (i0 + ii < Nv) cmac(acc[ii], d, qy[(i0 + ii) * n + k2]);
          }
#pragma unroll
          for (int ii = 0; ii < 8; ++ii)
            if (i0 + ii < Nv) W[(i0 + ii) * n + k] = acc[ii];
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < 8; ++m) {
          const int eh = t + 256 * m;
          if (eh < nh) {
            const int ic = eh / np, row = eh - ic * np;
            const int hr = row >= Nv ? 1 : 0, ir = row - hr * Nv;
            cx<double> acc = mk(0.0, 0.0);
            for (int k = hr * hn; k < (hr + 1) * hn; ++k) cjmac(acc, q[ir * (n + 1) + k], W[ic * n + k]);
            if (toX) accX[m] += acc;
            else accS[m] += acc;
          }
        }
      }
    }
  }
  cx<double>* out = Dn + ((long)A * 5 + kind) * nent;
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int eh = t + 256 * m;
    if (eh < nh) {
      const int e = hc * nh + eh;
      out[e] = accS[m] + accX[m];
      if (kind == 0) Xs[(long)A * nent + e] = accX[m];
    }
  }
}
template <class RQ>
void launch_assemble_coarse(const CGeom& cg, int Nv, int nagg, const int ab[4], const int* agg_sites,
                            const cx<double>* D, const cx<RQ>* Q, long qstride, cx<double>* Dn, cx<double>* Xs,
                            hipStream_t st) {
  size_t sm = (3 * (size_t)Nv * cg.n + Nv) * sizeof(cx<double>);
  if (Nv > 32) throw Error(INVALID_ARG, "coarse assembly supports Nv <= 32");
  hipLaunchKernelGGL(k_assemble_coarse<RQ>, dim3(10 * nagg), dim3(256), sm, st, cg, Nv, ab[0], ab[1], ab[2], ab[3],
                     agg_sites, D, Q, qstride, Dn, Xs);
}

// S += Gamma5 X^dag Gamma5 (self blocks, column-major), and S += X first when
// the assembly wrote the internal forward links to X only (add_x)
__global__ void k_self_fixup(int n, int nsites, cx<double>* __restrict__ D, const cx<double>* __restrict__ Xs,
                             int add_x) {
  long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  long nn = (long)n * n;
  if (gid >= (long)nsites * nn) return;
  int site = (int)(gid / nn);
  int e = (int)(gid - (long)site * nn);
  int col = e / n, row = e - col * n;
  cx<double> xv = Xs[(long)site * nn + (long)row * n + col];  // X(col,row)
  double s = g5(row, n) * g5(col, n);
  cx<double> d = D[(long)site * 5 * nn + e] + s * conj(xv);
  if (add_x) d += Xs[(long)site * nn + e];
  D[(long)site * 5 * nn + e] = d;
}
void launch_self_fixup(int n, int nsites, cx<double>* D, const cx<double>* Xs, int add_x, hipStream_t st) {
  long tot = (long)nsites * n * n;
  hipLaunchKernelGGL(k_self_fixup, dim3((tot + 255) / 256), dim3(256), 0, st, n, nsites, D, Xs, add_x);
}

// ---------------------------------------------------------------------------
// (S(c) + i tw Gamma5)^{-1} on the odd sites of the coarsest level: Gauss-Jordan
// with partial pivoting in FP64, one workgroup (64 threads) per odd site,
// working matrices in global scratch [nodd][2][n][n] (row-major A | inverse).
template <class R>
__global__ void __launch_bounds__(64) k_coarse_odd_inverse(CGeom cg, const cx<double>* __restrict__ D, double tw,
                                                           cx<double>* __restrict__ scr, cx<R>* __restrict__ Minv) {
  const int n = cg.n;
  const long nn = (long)n * n;
  int io = blockIdx.x;
  int site = cg.neven + io;
  int t = threadIdx.x;
  cx<double>* A = scr + (long)io * 2 * nn;
  cx<double>* Bm = A + nn;
  __shared__ cx<double> fcol[64];
  __shared__ int piv;
  if (t < n) {
    for (int r = 0; r < n; ++r) {
      cx<double> v = D[(long)site * 5 * nn + (long)t * n + r];  // element (r, t)
      if (r == t) v += mk(0.0, tw * g5(r, n));
      A[(long)r * n + t] = v;
      Bm[(long)r * n + t] = mk(r == t ? 1.0 : 0.0, 0.0);
    }
  }
  __syncthreads();
  for (int k = 0; k < n; ++k) {
    // pivot search over rows k..n-1 (thread t plays row t)
    double val = -1.0;
    int idx = k;
    if (t >= k && t < n) {
      val = norm2(A[(long)t * n + k]);
      idx = t;
    }
    for (int off = 32; off > 0; off >>= 1) {
      double ov = __shfl_xor(val, off, 64);
      int oi = __shfl_xor(idx, off, 64);
      if (ov > val || (ov == val && oi < idx)) {
        val = ov;
        idx = oi;
      }
    }
    if (t == 0) piv = idx;
    __syncthreads();
    int p = piv;
    if (t < n && p != k) {
      cx<double> a = A[(long)k * n + t], b = A[(long)p * n + t];
      A[(long)k * n + t] = b;
      A[(long)p * n + t] = a;
      a = Bm[(long)k * n + t];
      b = Bm[(long)p * n + t];
      Bm[(long)k * n + t] = b;
      Bm[(long)p * n + t] = a;
    }
    __syncthreads();
    cx<double> pv = A[(long)k * n + k];
    double d = norm2(pv);
    cx<double> inv = mk(pv.re / d, -pv.im / d);
    __syncthreads();
    if (t < n) {
      A[(long)k * n + t] = A[(long)k * n + t] * inv;
      Bm[(long)k * n + t] = Bm[(long)k * n + t] * inv;
      fcol[t] = A[(long)t * n + k];
    }
    __syncthreads();
    if (t < n) {
      cx<double> ak = A[(long)k * n + t], bk = Bm[(long)k * n + t];
      for (int r = 0; r < n; ++r) {
        if (r == k) continue;
        cx<double> f = fcol[r];
        A[(long)r * n + t] -= f * ak;
        Bm[(long)r * n + t] -= f * bk;
      }
    }
    __syncthreads();
  }
  if (t < n)
    for (int r = 0; r < n; ++r) {
      cx<double> v = Bm[(long)r * n + t];
      Minv[(long)io * nn + (long)t * n + r] = mk<R>((R)v.re, (R)v.im);  // column-major
    }
}
template <class R>
void launch_coarse_odd_inverse(const CGeom& cg, const cx<double>* D, double tw, cx<double>* scratch, cx<R>* Minv,
                               hipStream_t st) {
  int nodd = cg.nsites - cg.neven;
  hipLaunchKernelGGL(k_coarse_odd_inverse<R>, dim3(nodd), dim3(64), 0, st, cg, D, tw, scratch, Minv);
}

// ---------------------------------------------------------------------------
// odd sites: out = M (base - hop(in)) if base, else out = M hop(in)
template <class R, class S>
__global__ void __launch_bounds__(256) k_coarse_hop_inv_odd(CGeom cg,
                                                            const typename store_traits<S>::elem* __restrict__ D,
                                                            const cx<R>* __restrict__ Minv,
                                                            const cx<R>* __restrict__ in,
                                                            const cx<R>* __restrict__ base, cx<R>* __restrict__ out) {
  __shared__ cx<R> ys[4][9][64];
  __shared__ cx<R> us[4][64];
  int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int io = blockIdx.x * 4 + wv;
  int site = cg.neven + io;
  bool valid = site < cg.nsites;
  stage9(ys[wv], cg, site, valid, in, lane);
  __syncthreads();
  const int n = cg.n;
  if (valid && lane < n) {
    cx<R> u = hop_row<R, S>(cg, D, site, lane, ys[wv]);
    if (base) u = base[(long)site * n + lane] - u;
    us[wv][lane] = u;
  }
  __syncthreads();
  if (valid && lane < n) {
    const cx<R>* M = Minv + (long)io * n * n;
    cx<R> acc = mk<R>(0, 0);
    for (int l = 0; l < n; ++l) cmac(acc, M[(long)l * n + lane], us[wv][l]);
    out[(long)site * n + lane] = acc;
  }
}
// Whether the odd-even operator of one column on BF16 blocks goes to the matrix
// cores, as three columns that add up to it (FP16 blocks: the parts of an FP32 entry
// leave FP16's range).  us per pair, eight wavefronts on a site's rows and so: 32
// sites of n = 32 10.6 and 8.2, of n = 48 15.3 and 10.7; 1024 of n = 64 34.4 and
// 33.3; 4096 of n = 48 82.6 and 60.0.  n = 16 on more than 512 sites stays on the
// vector kernels (one_site: above 1024 sites, four to a workgroup).  Relative error of the full stencil against 64 bits, n = 16
// to 64: 9e-8 to 1.2e-7 there, 7e-8 here.
static inline bool one_mfma(int nsites, int n) { return n % 16 == 0 && (n > 16 || nsites <= 512); }
template <class R, class S>
void launch_coarse_hop_inv_odd(const CGeom& cg, const void* D, const cx<R>* Minv, const cx<R>* in, const cx<R>* base,
                               cx<R>* out, hipStream_t st) {
  const int nodd = cg.nsites - cg.neven;
  auto Dp = (const typename store_traits<S>::elem*)D;
  if constexpr (std::is_same<S, bf16>::value) {
    if (one_mfma(cg.nsites, cg.n)) return launch_coarse_hop_inv_odd_one<S>(cg, D, Minv, in, base, out, st);
  }
  if (one_site(nodd, cg.n))
    hipLaunchKernelGGL((k_coarse_hop_inv_odd_site<R, S>), dim3(nodd), dim3(SITE_T), 0, st, cg, Dp, Minv, in, base, out);
  else
    hipLaunchKernelGGL((k_coarse_hop_inv_odd<R, S>), dim3((nodd + 3) / 4), dim3(256), 0, st, cg, Dp, Minv, in, base,
                       out);
}

// even sites: mode 0: out = (S + i tw G5) v - hop(t);  mode 1: out = v - hop(t)
template <class R, class S>
__global__ void __launch_bounds__(256) k_coarse_schur_even(CGeom cg,
                                                           const typename store_traits<S>::elem* __restrict__ D, R tw,
                                                           const cx<R>* __restrict__ v, const cx<R>* __restrict__ tv,
                                                           cx<R>* __restrict__ out, int mode) {
  __shared__ cx<R> ys[4][9][64];
  __shared__ cx<R> vs[4][64];
  int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int site = blockIdx.x * 4 + wv;
  bool valid = site < cg.neven;
  stage9(ys[wv], cg, site, valid, tv, lane);
  const int n = cg.n;
  if (valid && lane < n) vs[wv][lane] = v[(long)site * n + lane];
  __syncthreads();
  if (valid && lane < n) {
    cx<R> acc = mode == 0 ? self_row<R, S>(cg, D, site, lane, tw, vs[wv]) : vs[wv][lane];
    acc -= hop_row<R, S>(cg, D, site, lane, ys[wv]);
    out[(long)site * n + lane] = acc;
  }
}
template <class R, class S>
void launch_coarse_schur_even(const CGeom& cg, const void* D, double tw, const cx<R>* v, const cx<R>* t, cx<R>* out,
                              int mode, hipStream_t st) {
  auto Dp = (const typename store_traits<S>::elem*)D;
  if constexpr (std::is_same<S, bf16>::value) {
    if (one_mfma(cg.nsites, cg.n)) return launch_coarse_schur_even_one<S>(cg, D, tw, v, t, out, mode, st);
  }
  if (one_site(cg.neven, cg.n))
    hipLaunchKernelGGL((k_coarse_schur_even_site<R, S>), dim3(cg.neven), dim3(SITE_T), 0, st, cg, Dp, (R)tw, v, t, out,
                       mode);
  else
    hipLaunchKernelGGL((k_coarse_schur_even<R, S>), dim3((cg.neven + 3) / 4), dim3(256), 0, st, cg, Dp, (R)tw, v, t,
                       out, mode);
}

// ---------------------------------------------------------------------------
#define INST_RS(R, S)                                                                                              \
  template void launch_coarse_apply<R, S>(const CGeom&, const void*, double, const cx<R>*, cx<R>*, hipStream_t);  \
  template void launch_coarse_residual<R, S>(const CGeom&, const void*, double, const cx<R>*, const cx<R>*,       \
                                             cx<R>*, hipStream_t);                                                \
  template void launch_coarse_sap<R, S>(const CGeom&, const void*, double, int, int, const int*, const int*,      \
                                        const cx<R>*, cx<R>*, int, hipStream_t);                                  \
  template void launch_coarse_sap_multi<R, S>(const CGeom&, const void*, double, int, int, const int*,            \
                                              const int*, const cx<R>*, cx<R>*, int, int, long, hipStream_t);     \
  template void launch_coarse_hop_inv_odd<R, S>(const CGeom&, const void*, const cx<R>*, const cx<R>*,            \
                                                const cx<R>*, cx<R>*, hipStream_t);                               \
  template void launch_coarse_schur_even<R, S>(const CGeom&, const void*, double, const cx<R>*, const cx<R>*,     \
                                               cx<R>*, int, hipStream_t);
INST_RS(double, double)
INST_RS(float, float)
INST_RS(float, f16)
INST_RS(float, bf16)

#define INST_R(R)                                                                                                   \
  template void launch_restrict_coarse<R>(int, int, int, int, const int*, const cx<R>*, long, const cx<R>*,        \
                                          cx<R>*, hipStream_t);                                                    \
  template void launch_prolong_coarse<R>(int, int, int, const int*, const cx<R>*, long, const cx<R>*, cx<R>*, int, \
                                         hipStream_t);                                                             \
  template void launch_restrict_coarse_m<R>(int, int, int, int, const int*, const cx<R>*, long, const cx<R>*, long, \
                                            cx<R>*, long, int, hipStream_t);                                       \
  template void launch_prolong_coarse_m<R>(int, int, int, const int*, const cx<R>*, long, const cx<R>*, long, cx<R>*, \
                                           long, int, int, hipStream_t);                                           \
  template void launch_qr_coarse<R, R>(int, int, int, int, const int*, const cx<R>*, long, cx<R>*, long, int*,   \
                                       hipStream_t);                                                               \
  template void launch_assemble_coarse<R>(const CGeom&, int, int, const int*, const int*, const cx<double>*,       \
                                          const cx<R>*, long, cx<double>*, cx<double>*, hipStream_t);              \
  template void launch_coarse_odd_inverse<R>(const CGeom&, const cx<double>*, double, cx<double>*, cx<R>*,         \
                                             hipStream_t);
INST_R(double)
INST_R(float)

}  // namespace ddamg
