"""K-column coarse operators of small and large grids, on the GPU: up to eight
columns take the kernels that split a site over four groups of wavefronts
(n = 64 on more than 512 sites per launch: one wavefront per 16 rows), more
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
                                     ((8, 8, 8, 32), 32),     # 1024 sites, n = 64: 512 per parity, split
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
