"""The network's training pass with its mixing layers and their adjoints on the
matrix cores, on the GPU against a plain torch complex128 reference (autograd):
both site counts per workgroup (16 below 32768 sites, 64 from there on), every
channel count that takes them, and the loss over several parts of an
aggregate's rows.  Tolerances are those of the network's other parity tests
(loss 1e-5, gradients 2e-4; the arithmetic is FP32)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

KAPPA, CSW, MU = 0.13729, 1.57551, 0.0009


def _transports(U, x):
    out = [x]
    for sign in (1, -1):
        for mu in range(4):
            u = U[..., mu, :, :]
            if sign > 0:
                f, m = torch.roll(x, -1, dims=1 + mu), u
            else:
                f, m = torch.roll(x, 1, dims=1 + mu), torch.roll(u, 1, dims=mu).mH.resolve_conj()
            out.append(sum(m[..., None, :, b] * f[..., b:b + 1] for b in range(3)))
    return torch.stack(out)


def _reference(U, x, W, a, b, Q, dims, block):
    """Loss and gradients (dL/dRe + i dL/dIm) by autograd in complex128."""
    C, V = x.shape[0], int(np.prod(dims))
    for l, w in enumerate(W):
        X = _transports(U, x).reshape(9, C, V, 4, 3).permute(0, 1, 3, 2, 4).reshape(9 * C * 4, V * 3)
        z = w.permute(1, 3, 0, 2, 4).reshape(C * 4, 9 * C * 4) @ X
        z = z.reshape(C, 4, V, 3).permute(0, 2, 1, 3).reshape((C,) + dims + (4, 3))
        if l < len(W) - 1:
            n = (z.real ** 2 + z.imag ** 2).sum(dim=(-1, -2))
            ex = (slice(None),) + (None,) * 4
            z = z * torch.sigmoid(a[l][ex] * n + b[l][ex])[..., None, None]
        x = z

    def halves(f):  # [blocks * 2, rows, C]
        nb = [d // c for d, c in zip(dims, block)]
        s = f.reshape(C, nb[0], block[0], nb[1], block[1], nb[2], block[2], nb[3], block[3], 2, 6)
        s = s.permute(1, 3, 5, 7, 9, 2, 4, 6, 8, 10, 0)
        return s.reshape(int(np.prod(nb)) * 2, -1, C).cpu()

    Y, T = halves(x), halves(Q)
    R = T - Y @ torch.linalg.solve(Y.mH @ Y, Y.mH @ T)
    loss = (R.real ** 2 + R.imag ** 2).sum() / (T.real ** 2 + T.imag ** 2).sum()
    loss.backward()
    return loss.item()


@pytest.mark.parametrize("C,L,dims,block", [(24, 3, (8, 8, 8, 8), (4, 4, 4, 4)),     # 16 sites per workgroup
                                            (16, 2, (4, 4, 4, 8), (2, 2, 2, 2)),     # aggregates of two tiles
                                            (8, 3, (4, 12, 4, 12), (2, 6, 2, 6)),    # 144 sites a block
                                            (8, 2, (16, 16, 16, 8), (4, 4, 4, 4))])  # 64 sites per workgroup
def test_training_pass(C, L, dims, block):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1611_01034_amd import ddamg, synth
    print(f"training pass: C {C}, L {L}, {dims}, {block}", flush=True)
    U = synth.gauge_field(dims, 0.3, 9101)
    W, a, b = synth.net_init_weights(C, L, 9102, scale=1.5)
    rng = np.random.default_rng(9103)
    a = [0.02 * rng.standard_normal(C) for _ in a]
    b = [0.5 * rng.standard_normal(C) for _ in b]
    noise = torch.from_numpy(synth.spinor(dims, 9104, nvec=C)).cuda()
    # orthonormal targets: QR per aggregate half
    nb = [d // c for d, c in zip(dims, block)]
    q = synth.gaussian((int(np.prod(nb)), 2, int(np.prod(block)) * 6, C), 9105)
    q = np.linalg.qr(q)[0].reshape(tuple(nb) + (2,) + tuple(block) + (6, C))
    Q = torch.from_numpy(np.ascontiguousarray(q.transpose(10, 0, 5, 1, 6, 2, 7, 3, 8, 4, 9))
                         .reshape((C,) + dims + (4, 3))).cuda()
    with ddamg.DDAMG(dims, block, KAPPA, CSW, MU, stream=torch.cuda.current_stream().cuda_stream) as ctx:
        ctx.set_gauge(U)
        ctx.net_create(L, C)
        ctx.net_set_params(ddamg.pack_net(W, a, b))
        loss, g = ctx.net_loss_grad(noise, Q)
        again, g2 = ctx.net_loss_grad(noise, Q)
    assert loss == again and np.array_equal(g, g2)
    Wt = [torch.from_numpy(w).cuda().requires_grad_() for w in W]
    at = [torch.from_numpy(v).cuda().requires_grad_() for v in a]
    bt = [torch.from_numpy(v).cuda().requires_grad_() for v in b]
    want = _reference(torch.from_numpy(U).cuda(), noise, Wt, at, bt, Q, dims, block)
    assert abs(loss - want) <= 1e-5 * want
    Wg, ag, bg = ddamg.unpack_net(g, C, L)
    rel = lambda u, v: np.linalg.norm(u - v) / np.linalg.norm(v)  # noqa: E731
    for l in range(L):
        assert rel(Wg[l], Wt[l].grad.resolve_conj().cpu().numpy()) < 2e-4, l
    for l in range(L - 1):
        assert rel(ag[l], at[l].grad.cpu().numpy()) < 2e-4 and rel(bg[l], bt[l].grad.cpu().numpy()) < 2e-4, l
