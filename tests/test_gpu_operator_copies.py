"""Reduced-precision copies of the fine operator (links, clover term, odd-site
inverses), on the GPU: a call makes the copies it reads and no others, and
each of them follows later changes of links, clover term, twist and boundary
phases.

Bars, fixed before the first run: device memory taken by the first call on a
new field is the copies' own size (links 36 entries of 8 or 4 bytes, clover
term 72 FP32 reals a site) plus one 64 MiB slab of the library's pool; results
after a change are the bits of a fresh context's, whose copies are made by the
same kernels from the same FP64 operator."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

KAPPA, CSW, MU = 0.13729, 1.57551, 0.0009


@pytest.fixture(scope="module")
def dd():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1611_01034_amd import ddamg
    return ddamg


def _ctx(dd, dims, block):
    return dd.DDAMG(dims, block, KAPPA, CSW, MU, stream=torch.cuda.current_stream().cuda_stream)


@pytest.mark.parametrize("prec,link_bytes", [("fp32", 8), ("fp16", 4), ("bf16", 4)])
def test_first_dirac_makes_the_copies_it_reads(dd, prec, link_bytes):
    """Neither the odd-site inverses (288 bytes a site) nor, for 16-bit links,
    the FP32 links (288) are made for D(mu)."""
    from paper_1611_01034_amd import synth
    dims, block = (32, 32, 16, 32), (4, 4, 4, 4)
    V = int(np.prod(dims))
    with _ctx(dd, dims, block) as ctx:
        ctx.set_gauge(synth.gauge_field_device(dims, 0.3, 8701))
        psi = synth.gaussian_device(dims + (4, 3), 8702)
        print(f"copies of the first D(mu): {prec}", flush=True)
        before = ctx.release_memory()
        ctx.apply_dirac(psi, precision=prec)
        taken = ctx.release_memory() - before
        assert taken <= V * (36 * link_bytes + 288) + (64 << 20), taken


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("dims,block", [((4, 4, 4, 4), (2, 2, 2, 2)),       # one tile of odd sites a block
                                        ((4, 12, 4, 12), (2, 6, 2, 6))])    # nine
def test_copies_follow_the_operator(dd, dims, block, prec):
    from oracle import dirac
    from paper_1611_01034_amd import synth
    U = [synth.gauge_field(dims, 0.3, 8801 + k) for k in range(2)]
    A = dirac.clover_blocks(dirac.WilsonClover(U[0], KAPPA, 1.2, MU).A)
    b, x0 = synth.spinor(dims, 8803), synth.spinor(dims, 8804)
    # each change, and whether the smoother has run before it
    changes = [("twist", lambda c: c.set_mu_eo(0.3, -0.45)), ("links", lambda c: c.set_gauge(U[1])),
               ("clover term", lambda c: c.set_clover(A)), ("phases", lambda c: c.set_boundary_phases((0.3, 0, 0, 0.1))),
               ("twist again", lambda c: c.set_mu(-0.2))]

    def both(c):
        return c.apply_dirac(b, precision=prec), c.sap(b, x0, iters=2, mr_steps=3, precision=prec)

    with _ctx(dd, dims, block) as ctx:
        ctx.set_gauge(U[0])
        ctx.apply_dirac(b, precision=prec)  # links and clover term, no inverses yet
        for n in range(1, len(changes) + 1):
            print(f"copies after {changes[n - 1][0]}: {dims} {block} {prec}", flush=True)
            changes[n - 1][1](ctx)
            got = both(ctx)
            with _ctx(dd, dims, block) as fresh:
                fresh.set_gauge(U[0])
                for _, f in changes[:n]:
                    f(fresh)
                want = both(fresh)
            for g, w in zip(got, want):
                assert np.array_equal(g, w), changes[n - 1][0]


@pytest.mark.parametrize("own,other", [("fp16", "bf16"), ("bf16", "fp16")])
def test_hierarchy_keeps_its_links(dd, own, other):
    """Calls in the other 16-bit type between two applications of a hierarchy's
    cycle leave it as it was: the same bits."""
    from paper_1611_01034_amd import synth
    dims, block = (8, 8, 8, 8), (4, 4, 4, 4)
    with _ctx(dd, dims, block) as ctx:
        ctx.set_gauge(synth.gauge_field(dims, 0.3, 8901))
        p = dd.default_params(levels=2, block=[block], nvec=[8], coarse_mu_factor=5.0, precision=own)
        ctx.set_test_vectors(p, [synth.spinor(dims, 8902, nvec=8)])
        b = synth.spinor(dims, 8903)
        first = ctx.vcycle(b)
        for call in (lambda: ctx.apply_dirac(b, precision=other), lambda: ctx.sap(b, b, 1, 4, other)):
            print(f"{own} hierarchy among {other} calls", flush=True)
            call()
            assert np.array_equal(ctx.vcycle(b), first)


def test_single_dirac_takes_no_memory(dd):
    """In place (out = in), on separate fields and on host fields: D(mu) of one
    field works in the context's own vectors, so it also runs when the device
    has no room for one more field."""
    import ctypes
    from paper_1611_01034_amd import synth
    dims, block = (32, 32, 16, 32), (4, 4, 4, 4)
    with _ctx(dd, dims, block) as ctx:
        ctx.set_gauge(synth.gauge_field_device(dims, 0.3, 8951))
        psi = synth.gaussian_device(dims + (4, 3), 8952)
        before = ctx.release_memory()
        want = ctx.apply_dirac(psi)
        print("one field on the host", flush=True)
        assert np.array_equal(ctx.apply_dirac(psi.cpu().numpy()), want.cpu().numpy())
        print("one field in place", flush=True)
        p = ctypes.c_void_p(psi.data_ptr())
        ctx._check(dd._lib.ddamg_apply_dirac(ctx._h, p, p, 1, dd.FP64, 1))
        assert torch.equal(psi, want)
        assert ctx.release_memory() == before
