"""K-column coarse operators of small and large grids, on the GPU: up to eight
columns take the kernels that split a site over four groups of wavefronts, more
columns the two-tile kernels.  The first columns of a 16-column application and
the same columns alone take different kernels on equally rounded inputs, so
they differ by the FP32 summation order only: 1e-5 of the norm of the
full stencil (9 n products of 2^-24 each, summed); 2e-4 for the odd-even
operator, whose second product rounds its input t to 16 bits (a difference of
1e-7 moves an entry of t across a rounding boundary, by 2^-8, once in about
2^-24 / 2^-9 cases: 2^-8 sqrt(2^-15) = 2e-5 of t, at most 2^3 larger in the
difference of the two products)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

KAPPA, CSW, MU = 0.13729, 1.57551, 0.0009


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
@pytest.mark.parametrize("dims,nv", [((4, 4, 4, 4), 8),       # 16 sites, n = 16
                                     ((8, 8, 8, 16), 16),     # 512 sites, n = 32
                                     ((8, 8, 8, 16), 24),     # n = 48
                                     ((8, 8, 8, 32), 32),     # 1024 sites, n = 64: 512 per parity
                                     ((8, 8, 16, 24), 32)])   # 1536 sites, n = 64: 768 per parity
def test_columns_alone_and_among_sixteen(dims, nv, prec):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1611_01034_amd import ddamg, synth
    block = (2, 2, 2, 2)
    with ddamg.DDAMG(dims, block, KAPPA, CSW, MU) as ctx:
        ctx.set_gauge(synth.gauge_field(dims, 0.3, 9201))
        p = ddamg.default_params(levels=2, block=[block], nvec=[nv], coarse_mu_factor=5.0, precision=prec)
        ctx.set_test_vectors(p, [synth.spinor(dims, 9202, nvec=nv)])
        cd, n = ctx.level_info(1)
        xs = synth.gaussian((16,) + cd + (n,), 9203)
        for name, tol in (("apply_coarse_multi", 1e-5), ("apply_coarse_schur_multi", 2e-4)):
            f = getattr(ctx, name)
            many = f(1, xs)
            for K in (1, 3, 8):
                print(f"{name}: {dims} n {n} {prec} K {K}", flush=True)
                got = f(1, xs[:K])
                for k in range(K):
                    d = np.linalg.norm(got[k] - many[k]) / np.linalg.norm(many[k])
                    assert d <= tol, (name, K, k, d)


def _round(x, prec):
    """Stored operator entries, rounded once to nearest even."""
    if prec == "fp64":
        return x
    if prec in ("fp32", "fp16"):
        t = np.float32 if prec == "fp32" else np.float16
        return x.real.astype(t).astype(np.float64) + 1j * x.imag.astype(t).astype(np.float64)

    def f(v):
        m, e = np.frexp(v)
        return np.ldexp(np.round(m * 256.0) / 256.0, e)
    return f(x.real) + 1j * f(x.imag)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("nv", [1, 4, 5, 9, 13, 16, 17, 26, 32])
def test_single_column_operators_of_any_width(nv, prec):
    """One workgroup per site (n = 2 .. 64: every split of the inner index, rows
    that 16-byte loads divide and rows that they do not) and, for n <= 24 on
    1536 sites, four sites per workgroup: D_c y and the odd-even operator
    against FP64 sums over the stored blocks.  FP64 1e-12; FP32 arithmetic 1e-5
    of the norm (9 n products of 2^-24 each; the odd-site inverse is held in
    FP32 and applied once more).  The odd-even operator of 16-bit storage runs
    here where n is no multiple of 16."""
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1611_01034_amd import ddamg, synth
    block = (2, 2, 2, 2)
    for dims in ((8, 8, 4, 4), (8, 8, 16, 24)) if nv <= 9 else ((8, 8, 4, 4),):
        with ddamg.DDAMG(dims, block, KAPPA, CSW, MU) as ctx:
            ctx.set_gauge(synth.gauge_field(dims, 0.3, 9301))
            p = ddamg.default_params(levels=2, block=[block], nvec=[nv], coarse_mu_factor=5.0, precision=prec)
            ctx.set_test_vectors(p, [synth.spinor(dims, 9302, nvec=nv)])
            cd, n = ctx.level_info(1)
            print(f"single column: {dims} n {n} {prec}", flush=True)
            S, F = (_round(a, prec) for a in ctx.get_coarse_op(1))
            y = synth.gaussian(cd + (n,), 9303)
            g = np.where(np.arange(n) < n // 2, -1.0, 1.0)
            tw = 5.0 * MU

            def hop(v):
                out = np.zeros_like(v)
                for mu in range(4):
                    out += (F[mu] @ np.roll(v, -1, axis=mu)[..., None])[..., 0]
                    Fb = np.conj(np.swapaxes(np.roll(F[mu], 1, axis=mu), -1, -2))
                    out += g * (Fb @ (g * np.roll(v, 1, axis=mu))[..., None])[..., 0]
                return out

            def site(v):
                return (S @ v[..., None])[..., 0] + 1j * tw * g * v

            tol = 1e-12 if prec == "fp64" else 1e-5
            want = site(y) + hop(y)
            got = ctx.apply_coarse(1, y)
            assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)
            if prec in ("fp16", "bf16") and n % 16 == 0:
                continue  # the K-column kernels, tested above
            par = np.indices(cd).sum(axis=0)[..., None] % 2
            Sd, _ = ctx.get_coarse_op(1)  # the inverse is that of the FP64 block
            u = np.linalg.solve(Sd + 1j * tw * np.diag(g), (par * hop((1 - par) * y))[..., None])[..., 0]
            want = (1 - par) * (site((1 - par) * y) - hop(u))
            got = ctx.apply_coarse_schur_multi(1, y[None])[0]
            assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)


@pytest.mark.parametrize("dims,nv", [((4, 4, 4, 4), 16), ((4, 4, 4, 8), 24), ((4, 4, 8, 8), 24), ((4, 4, 4, 4), 32)])
def test_even_rows_alone_on_few_sites(dims, nv):
    """16 rows of an even site to a workgroup (8 to 32 even sites, two to four row
    tiles): the columns alone against the same columns among sixteen, with the
    bars of the test above."""
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1611_01034_amd import ddamg, synth
    block = (2, 2, 2, 2)
    with ddamg.DDAMG(dims, block, KAPPA, CSW, MU) as ctx:
        ctx.set_gauge(synth.gauge_field(dims, 0.3, 9401))
        p = ddamg.default_params(levels=2, block=[block], nvec=[nv], coarse_mu_factor=5.0, precision="bf16")
        ctx.set_test_vectors(p, [synth.spinor(dims, 9402, nvec=nv)])
        cd, n = ctx.level_info(1)
        xs = synth.gaussian((16,) + cd + (n,), 9403)
        many = ctx.apply_coarse_schur_multi(1, xs)
        for K in (1, 5, 8):
            print(f"even rows: {dims} n {n} K {K}", flush=True)
            got = ctx.apply_coarse_schur_multi(1, xs[:K])
            for k in range(K):
                assert np.linalg.norm(got[k] - many[k]) <= 2e-4 * np.linalg.norm(many[k]), (K, k)


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
@pytest.mark.parametrize("dims,nv", [((4, 4, 4, 4), 8), ((4, 4, 4, 8), 16), ((4, 4, 8, 8), 24), ((8, 8, 8, 16), 32),
                                     ((8, 8, 8, 24), 16)])   # the last: 768 sites
def test_one_column_odd_even_solve(dims, nv, prec):
    """The coarsest solve of one column (BF16 blocks: the matrix cores, its FP32
    entries in three parts) to 1e-4, b on the even sites only: the
    even-site residual by the single-column stencil is that of the odd-even system,
    so 1e-4 of b and the 1e-5 of the FP32 operator.  Entries of b over twelve
    decades too.  (The accuracy of the operators themselves: test_gpu_one_column.py.)"""
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1611_01034_amd import ddamg, synth
    block = (2, 2, 2, 2)
    with ddamg.DDAMG(dims, block, KAPPA, CSW, MU) as ctx:
        ctx.set_gauge(synth.gauge_field(dims, 0.3, 9501))
        p = ddamg.default_params(levels=2, block=[block], nvec=[nv], coarse_mu_factor=5.0, precision=prec,
                                 coarse_tol=1e-4, coarse_max_iter=500, coarse_restart=30)
        ctx.set_test_vectors(p, [synth.spinor(dims, 9502, nvec=nv)])
        cd, n = ctx.level_info(1)
        even = 1 - np.indices(cd).sum(axis=0)[..., None] % 2
        b = even * synth.gaussian(cd + (n,), 9503)
        for v in (b, b * 10.0 ** np.random.default_rng(9504).uniform(-6, 6, b.shape)):
            print(f"one column: {dims} n {n} {prec}", flush=True)
            r = even * (v - ctx.apply_coarse(1, ctx.coarse_solve(1, v)))
            assert np.linalg.norm(r) <= 1.1e-4 * np.linalg.norm(v)
