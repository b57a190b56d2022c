// The fine operator D(+-mu) = D_W +- i Gamma5 mu (Sec. 1) on the whole
// lattice: Wilson hops with spin projection, the clover site term and the
// twist, in FP64 or FP32 arithmetic with FP64/FP32/FP16/BF16 link storage.
#include "finedev.hpp"

namespace ddamg {

// ---------------------------------------------------------------------------
// D(tw) psi, full lattice (tw: the twist of each parity), for K fields at a
// stride of ld complex.  One workgroup per (lattice block, field), one
// work-item per site; the block's input spinors are staged in LDS, so only
// hops that leave the block read neighbours from global memory.  The K
// fields of a block run in consecutive workgroups of one XCD, so the block's
// links and clover come from HBM once for all of them and from L2 for the
// rest.  With gm > 0 each XCD takes groups of gm consecutive blocks (two rows
// of blocks along X) while the XCDs sweep neighbouring groups together
// (group_remap); else each XCD sweeps one contiguous range of blocks
// (xcd_remap).
template <class R, class S>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 ? 2 : 3, 8)))
k_dirac(Geom g, int gm, const typename store_traits<S>::elem* __restrict__ U, const R* __restrict__ H, TwistR<R> tw,
        int K, long ld, const cx<R>* __restrict__ in, cx<R>* __restrict__ out) {
  extern __shared__ char smem_raw[];
  cx<R>* lds = reinterpret_cast<cx<R>*>(smem_raw);  // 12 x bs, parity-split
  const int w = gm > 0 ? group_remap(blockIdx.x, gm * K) : xcd_remap(blockIdx.x, gridDim.x), s = threadIdx.x;
  const int B = w / K, col = w - B * K;
  in += (long)col * ld;
  out += (long)col * ld;
  SiteNbr me;
  me_of(g, B, s, me);
  cx<R> psi[12], acc[12];
  load_spinor(in, g, B, s, psi);
#pragma unroll
  for (int c = 0; c < 12; ++c) *lds_site(lds, g, s, c) = psi[c];
  site_term(H, g, B, s, tw, psi, acc);
  __syncthreads();
  hop_staged<R, S>(U, in, lds, g, B, s, me, acc);
  // streaming stores: the result is not read again by this sweep, so it does
  // not need to take L2 from the halo lines of the blocks still running
  const long base = fidx(g, B, s, 12);
#pragma unroll
  for (int c = 0; c < 12; ++c) {
    __builtin_nontemporal_store(acc[c].re, &out[base + (long)c * TILE].re);
    __builtin_nontemporal_store(acc[c].im, &out[base + (long)c * TILE].im);
  }
}

template <class R, class S>
void launch_dirac_multi(const Geom& g, const void* U, const R* H, Twist tw, int K, long ld, const cx<R>* in,
                        cx<R>* out, hipStream_t st) {
  size_t sm = 12 * (size_t)g.bs * sizeof(cx<R>);
  const int gm = g.nblocks % (16 * g.nb[3]) == 0 ? 2 * g.nb[3] : 0;
  hipLaunchKernelGGL((k_dirac<R, S>), dim3(g.nblocks * K), dim3(g.bs), sm, st, g, gm,
                     (const typename store_traits<S>::elem*)U, H, TwistR<R>(tw), K, ld, in, out);
}
template <class R, class S>
void launch_dirac(const Geom& g, const void* U, const R* H, Twist tw, const cx<R>* in, cx<R>* out, hipStream_t st) {
  launch_dirac_multi<R, S>(g, U, H, tw, 1, 0, in, out, st);
}
#define DIRAC_INST(R, S)                                                                                     \
  template void launch_dirac<R, S>(const Geom&, const void*, const R*, Twist, const cx<R>*, cx<R>*, hipStream_t); \
  template void launch_dirac_multi<R, S>(const Geom&, const void*, const R*, Twist, int, long, const cx<R>*, cx<R>*, \
                                         hipStream_t);
DIRAC_INST(double, double)
DIRAC_INST(float, float)
DIRAC_INST(float, f16)
DIRAC_INST(float, bf16)
#undef DIRAC_INST

// ---------------------------------------------------------------------------
// The same operator between fields in the caller's layout (lexicographic
// [V][4][3] complex128), arithmetic in R: out = D(tw) in for K fields at a
// stride of ld complex, in one pass.  What bounds it is memory: the spinors
// are read and written once where a conversion to the block layout and back
// took two more passes each.  A block's sites are read as whole runs along X
// (consecutive threads read consecutive components) into LDS, rounded to R;
// in LDS a site's components lie together, padded to 13, so that both the
// staging writes and the per-site reads are free of bank conflicts.  A
// neighbour outside the block is read from the caller's field, where its 12
// components are contiguous (the block layout's X faces use two of every
// eight sites of a line).  The result goes back through the same LDS so that
// it too is written in whole runs.  The order of every sum is that of k_dirac.
// 64x32x32x32 FP64: 668 us (4.8 TB/s of 1536 B per site; conversions and
// k_dirac 338 + 738 + 390 us); six fields at 48x24x24x24: 893 us (2390).
constexpr int LEX_LS = 13;

template <class R>
__device__ __forceinline__ void load_nbr_lex(const cx<double>* in, const cx<R>* lds, int B, int Bn, int sn, int ln,
                                             cx<R> p[12]) {
  if (Bn == B) {
#pragma unroll
    for (int c = 0; c < 12; ++c) p[c] = lds[sn * LEX_LS + c];
  } else {
    const cx<double>* q = in + (long)ln * 12;
#pragma unroll
    for (int c = 0; c < 12; ++c) p[c] = mk<R>((R)q[c].re, (R)q[c].im);
  }
}

template <int MU, class R, class S>
__device__ __forceinline__ void hop_lex_dir(const typename store_traits<S>::elem* U, const cx<double>* in,
                                            const cx<R>* lds, const Geom& g, int B, int s, const SiteNbr& me, int lex,
                                            cx<R> out[12]) {
  cx<R> psi[12], u[9];
  int Bn, sn;
  int str = 1;  // lexicographic stride of direction MU
#pragma unroll
  for (int d = MU + 1; d < 4; ++d) str *= g.L[d];
  const int wrap = (g.L[MU] - 1) * str;
  nbr_of(g, me, MU, +1, Bn, sn);
  const bool hi = me.l[MU] == g.b[MU] - 1 && me.bc[MU] == g.nb[MU] - 1;
  load_nbr_lex(in, lds, B, Bn, sn, hi ? lex - wrap : lex + str, psi);
  load_link_t<MU, R, S>(U, g, B, s, u);
  hop_accum_t<0, MU>(psi, u, out);
  nbr_of(g, me, MU, -1, Bn, sn);
  const bool lo = me.l[MU] == 0 && me.bc[MU] == 0;
  load_nbr_lex(in, lds, B, Bn, sn, lo ? lex + wrap : lex - str, psi);
  load_link_t<MU, R, S>(U, g, Bn, sn, u);
  hop_accum_t<1, MU>(psi, u, out);
}

template <class R, class S>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 ? 2 : 3, 8)))
k_dirac_lex(Geom g, int gm, const typename store_traits<S>::elem* __restrict__ U, const R* __restrict__ H,
            TwistR<R> tw, int K, long ld, const cx<double>* __restrict__ in, cx<double>* __restrict__ out) {
  typedef double v2d __attribute__((ext_vector_type(2)));
  extern __shared__ char smem_raw[];
  cx<R>* lds = reinterpret_cast<cx<R>*>(smem_raw);  // bs x LEX_LS
  __shared__ int xof[256], sof[256];                // lexicographic site and slot of the block's j-th site
  const int w = gm > 0 ? group_remap(blockIdx.x, gm * K) : xcd_remap(blockIdx.x, gridDim.x), s = threadIdx.x;
  const int B = w / K, col = w - B * K;
  in += (long)col * ld;
  out += (long)col * ld;
  SiteNbr me;
  me_of(g, B, s, me);
  int lex;
  {
    int x[4];
    for (int d = 0; d < 4; ++d) x[d] = me.bc[d] * g.b[d] + me.l[d];
    lex = (int)lex_index(g, x);
    const int j = ((me.l[0] * g.b[1] + me.l[1]) * g.b[2] + me.l[2]) * g.b[3] + me.l[3];
    xof[j] = lex;
    sof[j] = s;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const int e = i * g.bs + s, j = e / 12, c = e - 12 * j;
    const cx<double> v = in[(long)xof[j] * 12 + c];
    lds[sof[j] * LEX_LS + c] = mk<R>((R)v.re, (R)v.im);
  }
  __syncthreads();
  cx<R> psi[12], acc[12];
#pragma unroll
  for (int c = 0; c < 12; ++c) psi[c] = lds[s * LEX_LS + c];
  site_term(H, g, B, s, tw, psi, acc);
#pragma unroll 1
  for (int mu = 0; mu < g.ndir; ++mu) {
    switch (mu) {
      case 0: hop_lex_dir<0, R, S>(U, in, lds, g, B, s, me, lex, acc); break;
      case 1: hop_lex_dir<1, R, S>(U, in, lds, g, B, s, me, lex, acc); break;
      case 2: hop_lex_dir<2, R, S>(U, in, lds, g, B, s, me, lex, acc); break;
      default: hop_lex_dir<3, R, S>(U, in, lds, g, B, s, me, lex, acc); break;
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 12; ++c) lds[s * LEX_LS + c] = acc[c];
  __syncthreads();
  // streaming stores, as in k_dirac
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const int e = i * g.bs + s, j = e / 12, c = e - 12 * j;
    const cx<R> v = lds[sof[j] * LEX_LS + c];
    __builtin_nontemporal_store(v2d{(double)v.re, (double)v.im},
                                reinterpret_cast<v2d*>(out + (long)xof[j] * 12 + c));
  }
}

template <class R, class S>
void launch_dirac_lex(const Geom& g, const void* U, const R* H, Twist tw, int K, long ld, const cx<double>* in,
                      cx<double>* out, hipStream_t st) {
  if (g.V > 0x7fffffffL) throw Error(INVALID_ARG, "lattice of 2^31 sites or more");
  const size_t sm = (size_t)LEX_LS * g.bs * sizeof(cx<R>);
  const int gm = g.nblocks % (16 * g.nb[3]) == 0 ? 2 * g.nb[3] : 0;
  hipLaunchKernelGGL((k_dirac_lex<R, S>), dim3(g.nblocks * K), dim3(g.bs), sm, st, g, gm,
                     (const typename store_traits<S>::elem*)U, H, TwistR<R>(tw), K, ld, in, out);
}
#define LEX_INST(R, S)                                                                                            \
  template void launch_dirac_lex<R, S>(const Geom&, const void*, const R*, Twist, int, long, const cx<double>*, \
                                       cx<double>*, hipStream_t);
LEX_INST(double, double)
LEX_INST(float, float)
LEX_INST(float, f16)
LEX_INST(float, bf16)
#undef LEX_INST

}  // namespace ddamg
