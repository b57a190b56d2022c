"""The odd-even coarse operator of one column against FP64, on the GPU.  BF16
blocks with n a multiple of 16 take the matrix cores (an FP32 entry in three
parts; n = 16 on up to 512 sites only), the others the vector kernels: a
workgroup per site, or on more than 512 sites of a parity and n <= 24 four
sites to a workgroup.

Two GMRES steps of the coarsest solve from zero show the operator's own
accuracy: x_e lies in the span of r and A r, with r = b_e - D_eo D_oo^-1 b_o
and A the odd-even operator, and x_o = D_oo^-1 (b_o - D_oe x_e).  Both are
compared with FP64 over the stored blocks, for b on all sites (r comes from the
kernels) and on the even ones (x_o is nothing but hops of x_e).

Bar, fixed before the first run: 6e-7 of the norm.  In a model of the path in
numpy (16 to 128 sites, n = 16 to 64) FP32 sums of the exact products leave 0.8e-7 to
1.4e-7; with the third part of the entries left out 2.2e-6 to 2.7e-6 (x_o of b on all
sites, where b_o hides most of it: 0.3e-6 to 0.6e-6).  The bar is the geometric mean
of the two."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

KAPPA, CSW, MU = 0.13729, 1.57551, 0.0009
BAR = 6e-7


def _round(x, prec):
    """Stored operator entries, rounded once to nearest even."""
    if prec == "fp16":
        return x.real.astype(np.float16).astype(np.float64) + 1j * x.imag.astype(np.float16).astype(np.float64)

    def f(v):
        m, e = np.frexp(v)
        return np.ldexp(np.round(m * 256.0) / 256.0, e)
    return f(x.real) + 1j * f(x.imag)


class _OddEven:
    """FP64 odd-even operator over the stored blocks S, F; the odd-site inverse
    is that of the unrounded site block."""

    def __init__(self, S, F, tw, prec):
        n = S.shape[-1]
        self.g = np.where(np.arange(n) < n // 2, -1.0, 1.0)
        self.tw = tw
        self.M = S + 1j * tw * np.diag(self.g)
        self.S, self.F = _round(S, prec), [_round(F[mu], prec) for mu in range(4)]
        self.odd = np.indices(S.shape[:4]).sum(axis=0)[..., None] % 2
        self.even = 1 - self.odd

    def hop(self, v):
        out = np.zeros_like(v)
        for mu in range(4):
            out += (self.F[mu] @ np.roll(v, -1, axis=mu)[..., None])[..., 0]
            Fb = np.conj(np.swapaxes(np.roll(self.F[mu], 1, axis=mu), -1, -2))
            out += self.g * (Fb @ (self.g * np.roll(v, 1, axis=mu))[..., None])[..., 0]
        return out

    def inv(self, v):
        return np.linalg.solve(self.M, (self.odd * v)[..., None])[..., 0]

    def rhs(self, b):
        return self.even * (b - self.hop(self.inv(b)))

    def schur(self, v):
        site = (self.S @ v[..., None])[..., 0] + 1j * self.tw * self.g * v
        return self.even * (site - self.hop(self.inv(self.hop(v))))


@pytest.mark.parametrize("dims,nv,prec", [
    ((4, 4, 4, 4), 8, "bf16"), ((4, 4, 4, 4), 16, "bf16"),      # 16 sites: 16 rows of an even site a workgroup
    ((4, 4, 4, 4), 24, "bf16"), ((4, 4, 4, 4), 32, "bf16"),
    ((8, 8, 8, 16), 8, "bf16"), ((8, 8, 8, 16), 16, "bf16"),    # 512 sites: a workgroup per even site
    ((8, 8, 8, 16), 24, "bf16"), ((8, 8, 8, 16), 32, "bf16"),
    ((8, 8, 8, 24), 8, "bf16"), ((8, 8, 8, 24), 16, "bf16"),    # 768 sites: n = 16 on the vector kernels, 32 not
    ((8, 8, 16, 24), 8, "bf16"),                                # 1536 sites: four to a workgroup
    ((4, 4, 4, 4), 16, "fp16"), ((8, 8, 16, 24), 8, "fp16")])   # FP16 blocks: vector kernels
def test_one_column_against_fp64(dims, nv, prec):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1611_01034_amd import ddamg, synth
    block = (2, 2, 2, 2)
    with ddamg.DDAMG(dims, block, KAPPA, CSW, MU) as ctx:
        ctx.set_gauge(synth.gauge_field(dims, 0.3, 9701))
        p = ddamg.default_params(levels=2, block=[block], nvec=[nv], coarse_mu_factor=5.0, precision=prec,
                                 coarse_restart=2, coarse_max_iter=2, coarse_tol=1e-30)
        ctx.set_test_vectors(p, [synth.spinor(dims, 9702, nvec=nv)])
        cd, n = ctx.level_info(1)
        S, F = ctx.get_coarse_op(1)
        op = _OddEven(S, F, 5.0 * MU, prec)
        b = synth.gaussian(cd + (n,), 9703)
        for name, v in (("all sites", b), ("even sites", op.even * b)):
            print(f"one column: {dims} n {n} {prec}, b on {name}", flush=True)
            x = ctx.coarse_solve(1, v)
            xe, xo = op.even * x, op.odd * x
            want = op.inv(v - op.hop(xe))
            assert np.linalg.norm(xo - want) <= BAR * np.linalg.norm(want)
            r = op.rhs(v)
            q = np.linalg.qr(np.stack([r.ravel(), op.schur(r).ravel()], axis=1))[0]
            u = xe.ravel()
            assert np.linalg.norm(u - q @ (q.conj().T @ u)) <= BAR * np.linalg.norm(u)
