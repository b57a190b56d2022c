"""Kernels that read and write the caller's lexicographic fields, on the GPU
against the oracle (FP64, Sec. 1 D(mu)): blocks and extents that are no powers
of two, both block orders of the launch, several fields, every precision, and
fields that overlap.

Tolerances, fixed before the first run: FP64 1e-12 of the result (the FP64
operator bar); FP32 arithmetic 2e-6 (eight hops of 3-term complex sums and a
6-term site term, each rounded once to 2^-24, on results of order 10 times an
entry); FP16 / BF16 links the same against the oracle on links rounded the
same way."""
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


def _case(dd, dims, block, seed, mu_odd=None):
    from oracle import dirac
    from paper_1611_01034_amd import synth
    U = synth.gauge_field(dims, 0.3, seed)
    ctx = dd.DDAMG(dims, block, KAPPA, CSW, MU, stream=torch.cuda.current_stream().cuda_stream)
    ctx.set_gauge(U)
    return ctx, U, dirac.WilsonClover(U, KAPPA, CSW, MU)


def _round_links(U, prec):
    """Links rounded once to nearest even (no intermediate FP32)."""
    if prec == "fp16":
        f = lambda v: v.astype(np.float16).astype(np.float64)
    else:
        def f(v):
            m, e = np.frexp(v)
            return np.ldexp(np.round(m * 256.0) / 256.0, e)
    return f(U.real) + 1j * f(U.imag)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16", "bf16"])
@pytest.mark.parametrize("dims,block", [((4, 4, 4, 4), (2, 2, 2, 2)),      # 16 sites a block, one row of two blocks
                                        ((4, 12, 4, 12), (2, 6, 2, 6)),    # 144 sites, two wavefronts and a quarter
                                        ((8, 4, 12, 8), (4, 2, 6, 4)),     # 192 sites
                                        ((8, 8, 8, 16), (4, 4, 4, 4))])    # 256 sites, the other block order
def test_dirac_on_caller_fields(dd, dims, block, prec):
    from oracle import dirac
    from paper_1611_01034_amd import synth
    ctx, U, op = _case(dd, dims, block, 8101)
    try:
        print(f"D(mu) on caller fields: {dims} {block} {prec}", flush=True)
        K = 3
        psi = synth.spinor(dims, 8102, nvec=K)
        dev = torch.from_numpy(psi).cuda()
        one = [ctx.apply_dirac(dev[k].clone(), precision=prec) for k in range(K)]
        many = ctx.apply_dirac_multi(dev, sign=+1, precision=prec)
        host = ctx.apply_dirac(psi[1], precision=prec)
        ref_op = op
        if prec in ("fp16", "bf16"):
            ref_op = dirac.WilsonClover(_round_links(U, prec), KAPPA, CSW, MU, clover=dirac.clover_blocks(op.A))
        tol = 1e-12 if prec == "fp64" else 2e-6
        for k in range(K):
            ref = ref_op.apply(psi[k])
            got = one[k].cpu().numpy()
            assert np.linalg.norm(got - ref) <= tol * np.linalg.norm(ref)
            assert torch.equal(one[k], many[k])
        assert np.array_equal(host, one[1].cpu().numpy())
    finally:
        ctx.close()


@pytest.mark.parametrize("shift", [0, 1, 12])
def test_dirac_with_overlapping_fields(dd, shift):
    """out over in (shifted by `shift` complex entries): as on separate fields."""
    import ctypes
    from paper_1611_01034_amd import synth
    dims, block = (8, 4, 12, 8), (4, 2, 6, 4)
    ctx, _, _ = _case(dd, dims, block, 8201)
    try:
        n = int(np.prod(dims)) * 12
        psi = torch.from_numpy(synth.spinor(dims, 8202)).cuda()
        ref = ctx.apply_dirac(psi)
        for entry in ("apply_dirac", "noalloc"):
            print(f"overlapping fields: shift {shift}, {entry}", flush=True)
            buf = torch.zeros(n + shift, dtype=torch.complex128, device="cuda")
            buf[:n] = psi.reshape(-1)
            pi = ctypes.c_void_p(buf.data_ptr())
            po = ctypes.c_void_p(buf.data_ptr() + 16 * shift)
            torch.cuda.synchronize()
            if entry == "noalloc":
                ctx._check(dd._lib.ddamg_apply_dirac_noalloc(ctx._h, pi, po, 1))
            else:
                ctx._check(dd._lib.ddamg_apply_dirac(ctx._h, pi, po, 1, dd.FP64, 1))
            torch.cuda.synchronize()
            assert torch.equal(buf[shift:].reshape(ref.shape), ref)
    finally:
        ctx.close()


@pytest.mark.parametrize("dims,block", [((4, 4, 4, 4), (2, 2, 2, 2)), ((4, 12, 4, 12), (2, 6, 2, 6)),
                                        ((8, 4, 12, 8), (4, 2, 6, 4))])
def test_new_field_on_ragged_blocks(dd, dims, block):
    """Clover term and odd-site inverses of a new field (set twice: nothing of
    the first one stays): the clover blocks within 1e-13, and one FP64 SAP
    iteration, which applies T_oo^-1 in every step, within 1e-11 of the oracle
    (the bars of the parity tests)."""
    from oracle import dirac, sap, stencil
    from paper_1611_01034_amd import synth
    ctx, _, _ = _case(dd, dims, block, 8301)
    try:
        print(f"new field: {dims} {block}", flush=True)
        U = synth.gauge_field(dims, 0.4, 8302)
        ctx.set_mu(0.05)
        ctx.set_gauge(U)
        op = dirac.WilsonClover(U, KAPPA, CSW, 0.05)
        assert np.abs(ctx.get_clover() - dirac.clover_blocks(op.A)).max() < 1e-13
        b = synth.spinor(dims, 8303)
        got = ctx.sap(b, np.zeros_like(b), iters=1, mr_steps=3)
        want = sap.sap(stencil.FineLevel(op), b.reshape(dims + (12,)), np.zeros(dims + (12,), complex), block, 3, 1)
        assert np.linalg.norm(got.reshape(want.shape) - want) <= 1e-11 * np.linalg.norm(want)
    finally:
        ctx.close()


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("dims,block", [((4, 4, 4, 4), (2, 2, 2, 2)), ((4, 12, 4, 12), (2, 6, 2, 6)),
                                        ((8, 4, 12, 8), (4, 2, 6, 4))])
def test_layout_conversions_of_several_fields(dd, dims, block, prec):
    """Device fields (all of them converted by one launch) against host fields
    (one at a time): zero SAP iterations give x back, rounded once to the
    arithmetic; two iterations the same bits; FP64 within 1e-11 of the oracle."""
    import ctypes
    from oracle import sap, stencil
    from paper_1611_01034_amd import synth
    ctx, U, op = _case(dd, dims, block, 8401)
    try:
        print(f"layout conversions: {dims} {block} {prec}", flush=True)
        K = 3
        b, x0 = synth.spinor(dims, 8402, nvec=K), synth.spinor(dims, 8403, nvec=K)
        db = torch.from_numpy(b).cuda()
        for iters in (0, 2):
            x = torch.from_numpy(x0).cuda()
            ctx._check(dd._lib.ddamg_sap_multi(ctx._h, K, ctypes.c_void_p(db.data_ptr()),
                                               ctypes.c_void_p(x.data_ptr()), iters, 3, dd.PRECISIONS[prec], 1))
            host = ctx.sap_multi(b, x0, iters, 3, prec)
            assert np.array_equal(x.cpu().numpy(), host)
            if iters == 0:
                want = x0 if prec == "fp64" else x0.astype(np.complex64).astype(np.complex128)
                assert np.array_equal(host, want)
            elif prec == "fp64":
                fl = stencil.FineLevel(op)
                for k in range(K):
                    want = sap.sap(fl, b[k].reshape(dims + (12,)), x0[k].reshape(dims + (12,)), block, 3, 2)
                    assert np.linalg.norm(host[k].reshape(want.shape) - want) <= 1e-11 * np.linalg.norm(want)
    finally:
        ctx.close()


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("dims,block", [((4, 4, 4, 4), (2, 2, 2, 2)), ((4, 12, 4, 12), (2, 6, 2, 6)),
                                        ((8, 4, 12, 8), (4, 2, 6, 4))])
def test_reduced_precision_sap_after_twist_changes(dd, dims, block, prec):
    """The FP32 odd-site inverses follow the odd sites' twist: sweeps at the
    first twist, at different twists on the two parities and at a negative one,
    each within 1e-5 of the oracle on links rounded the same way (the FP32 SAP
    bar of the parity tests)."""
    from oracle import dirac, sap, stencil
    from paper_1611_01034_amd import synth
    ctx, U, _ = _case(dd, dims, block, 8501)
    try:
        print(f"sap after twist changes: {dims} {block} {prec}", flush=True)
        Ur = U.astype(np.complex64).astype(np.complex128) if prec == "fp32" else _round_links(U, prec)
        # the clover term comes from the links as given
        A = dirac.clover_blocks(dirac.WilsonClover(U, KAPPA, CSW, 0.0).A)
        b, x0 = synth.spinor(dims, 8502), synth.spinor(dims, 8503)
        for mu, mu_odd in ((MU, MU), (0.3, -0.45), (-0.2, -0.2)):
            ctx.set_mu(mu) if mu == mu_odd else ctx.set_mu_eo(mu, mu_odd)
            got = ctx.sap(b, x0, iters=2, mr_steps=3, precision=prec)
            op = dirac.WilsonClover(Ur, KAPPA, CSW, mu, clover=A, mu_odd=mu_odd)
            want = sap.sap(stencil.FineLevel(op), b.reshape(dims + (12,)), x0.reshape(dims + (12,)), block, 3, 2)
            assert np.linalg.norm(got.reshape(want.shape) - want) <= 1e-5 * np.linalg.norm(want), (mu, mu_odd)
    finally:
        ctx.close()


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("dims,block,K", [((4, 12, 8, 24), (2, 6, 2, 6), 16),     # 32 workgroups a field: 128 wavefronts
                                          ((8, 4, 24, 8), (4, 2, 6, 4), 16),      # 16 workgroups: 64, and 1024 together
                                          ((8, 8, 16, 24), (2, 2, 2, 2), 2)])     # 768 workgroups: 1536 wavefronts
def test_sap_on_few_and_many_blocks(dd, dims, block, K, prec):
    """A sweep of few workgroups (and of one field with FP32 links on many) gives
    two threads to a pair of slots, the others one: K fields in one call against
    one at a time, each within 1e-5 of the exact sweep, so 2e-5 apart.  n_MR = 0
    too, where only the odd sites move."""
    from paper_1611_01034_amd import synth
    ctx, _, _ = _case(dd, dims, block, 8601)
    try:
        print(f"sap few and many: {dims} {block} {K} {prec}", flush=True)
        b, x0 = synth.spinor(dims, 8602, nvec=K), synth.spinor(dims, 8603, nvec=K)
        for n_mr in (0, 3):
            many = ctx.sap_multi(b, x0, 2, n_mr, prec)
            for k in (0, K - 1):
                one = ctx.sap(b[k], x0[k], 2, n_mr, prec)
                assert np.linalg.norm(one - many[k]) <= 2e-5 * np.linalg.norm(many[k]), (n_mr, k)
    finally:
        ctx.close()
