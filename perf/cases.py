"""Workloads of the library: what programs that use it call, at the sizes and
options they call it with.

    listed()            the named cases
    draw(rng)           one more case of the same ranges
    prepare(case, seed) what a program holds before the call, on the GPU
    run(state)          one pass through the public entry points
    work(case)          bytes and operations a pass cannot do without
    exact(case, seed)   the values of a pass in 64 bits, by plain torch

The physics is that of the bench: links exp(i eps H) with eps = 0.3,
kappa = 0.13729, c_sw = 1.57551, mu = 0.0009, Gaussian sources.

Fields that the library computes in FP32 arithmetic come back from it widened
to complex128; a program that asked for such a precision keeps them as
complex64 (nothing is lost: every value is an FP32 number), so these cases
return complex64.  What is computed in FP64 is returned in complex128.
"""
import ctypes

import numpy as np
import torch

from paper_1611_01034_amd import ddamg, synth

KAPPA, CSW, MU, EPS = 0.13729, 1.57551, 0.0009, 0.3
DELTA = 5.0
# HMC acceptance tests ask for solutions near the limit of FP64
TOL = 1e-12


def listed():
    return [
        # one D(mu) on the quick-start lattice: the smallest call, all latency
        dict(name="dirac_8x8x8x16_fp64", op="dirac", dims="8,8,8,16", block="4,4,4,4", precision="fp64"),
        # D(mu) on a lattice that fills the card: residual checks, measurements
        dict(name="dirac_64x32x32x32_fp64", op="dirac", dims="64,32,32,32", block="4,4,4,4", precision="fp64"),
        # reduced-precision D(mu) with blocks and extents that are no powers of two
        dict(name="dirac_20x12x12x24_bf16", op="dirac", dims="20,12,12,24", block="2,6,2,6", precision="bf16"),
        # D(mu) on the six columns of a lock-step group, as block Krylov methods call it
        dict(name="dirac6_48x24x24x24_fp64", op="dirac_multi", dims="48,24,24,24", block="4,4,4,4", precision="fp64",
             nfields=6),
        # the smoother on the six columns of a lock-step group, the mixed form's precision
        dict(name="sap6_48x24x24x24_bf16", op="sap", dims="48,24,24,24", block="4,4,4,4", precision="bf16", nfields=6,
             iters=2, mr_steps=4),
        # the smoother on one field in FP32
        dict(name="sap_24x16x16x24_fp32", op="sap", dims="24,16,16,24", block="4,4,4,4", precision="fp32", nfields=1,
             iters=3, mr_steps=4),
        # a new gauge field of an HMC trajectory (links, clover term, odd-site inverses) and its first D(mu)
        dict(name="field_48x24x24x24", op="field", dims="48,24,24,24", block="4,4,4,4"),
        # the quick start: a two-level solve of one source with the setup in hand
        dict(name="solve_8x8x8x16_bf16", op="solve", dims="8,8,8,16", block="4,4,4,4", levels=2, nvec=16, nvec2=0,
             precision="bf16", nrhs=1, rhs_batch=1, sap_post=3, restart=10),
        # 12 sources (a point source's spins and colours) in lock-step groups of 6, as the bench solves them
        dict(name="solve12_16x16x16x32_bf16", op="solve", dims="16,16,16,32", block="4,4,4,4", levels=2, nvec=24,
             nvec2=0, precision="bf16", nrhs=12, rhs_batch=6, sap_post=2, restart=10),
        # the bench's step (setup with one iteration, then the sources)
        dict(name="setup_solve6_32x32x32x32_bf16", op="setup_solve", dims="32,32,32,32", block="4,4,4,4", levels=3,
             nvec=24, nvec2=32, precision="bf16", nrhs=6, rhs_batch=6, sap_post=2, restart=4),
        # the setup's network: inference on a production-like lattice
        dict(name="net_forward_32x16x16x16", op="net_forward", dims="32,16,16,16", block="4,4,4,4", layers=4, chan=24),
        # the setup's network: loss and gradient of a training step
        dict(name="net_grad_8x8x8x8", op="net_grad", dims="8,8,8,8", block="4,4,4,4", layers=4, chan=24),
    ]


_BLOCKS = [(4, 4, 4, 4), (4, 4, 4, 4), (4, 4, 4, 4), (2, 2, 2, 2), (2, 4, 4, 6), (2, 6, 2, 6), (4, 2, 6, 4)]


def _txt(v):
    return ",".join(str(int(x)) for x in v)


def _dims(rng, block, lo, hi, mult=2):
    """Extents with a number of blocks per direction that is a multiple of
    `mult`, the volume spread over the logarithm of lo..hi."""
    want = lo * (hi / lo) ** rng.random()
    unit = [mult * b for b in block]
    d = list(unit)
    for _ in range(400):
        v = d[0] * d[1] * d[2] * d[3]
        if v >= want:
            break
        i = rng.randrange(4)
        if v // d[i] * (d[i] + unit[i]) > hi:
            break
        if d[i] + unit[i] <= 96:
            d[i] += unit[i]
    return d


def draw(rng):
    op = rng.choice(["dirac", "dirac", "dirac_noalloc", "dirac_multi", "sap", "sap", "field", "solve", "solve",
                     "setup_solve", "net_forward", "net_grad"])
    prec = rng.choice(["fp64", "fp32", "fp16", "bf16"])
    block = rng.choice(_BLOCKS)
    if op == "dirac":
        return dict(op=op, dims=_txt(_dims(rng, block, 4096, 2000000)), block=_txt(block), precision=prec)
    if op == "dirac_noalloc":
        return dict(op=op, dims=_txt(_dims(rng, block, 4096, 131072)), block=_txt(block), precision="fp64")
    if op == "dirac_multi":
        k = rng.randint(2, 12)
        return dict(op=op, dims=_txt(_dims(rng, block, 4096, 3900000 // k)), block=_txt(block), precision=prec,
                    nfields=k)
    if op == "sap":
        k = rng.randint(1, 12)
        return dict(op=op, dims=_txt(_dims(rng, block, 4096, 1000000 // k)), block=_txt(block), precision=prec,
                    nfields=k, iters=rng.randint(1, 3), mr_steps=rng.randint(2, 5))
    if op == "field":
        return dict(op=op, dims=_txt(_dims(rng, block, 4096, 600000)), block=_txt(block))
    if op == "net_forward":
        return dict(op=op, dims=_txt(_dims(rng, (4, 4, 4, 4), 4096, 60000)), block="4,4,4,4",
                    layers=rng.randint(2, 4), chan=rng.choice([4, 8, 12, 16, 24]))
    if op == "net_grad":
        return dict(op=op, dims=_txt(_dims(rng, (4, 4, 4, 4), 4096, 8192)), block="4,4,4,4",
                    layers=rng.randint(2, 4), chan=rng.choice([4, 8, 12, 16, 24]))
    if rng.random() < 0.4:
        # three levels need extents that are multiples of 16; with fewer test
        # vectors such a small lattice needs many times the iterations
        dims, levels, nvec, nvec2 = (16, 16, 16, 16), 3, 24, 32
        prec = rng.choice(["fp16", "bf16", "bf16"])
        k = rng.randint(2, 6)
        kb = rng.randint(2, k)
    else:
        dims, levels = _dims(rng, (4, 4, 4, 4), 4096, 20000 if prec == "fp64" else 50000), 2
        nvec, nvec2 = rng.choice([16, 20, 24]), 0
        k = rng.randint(1, 3 if prec in ("fp64", "fp32") else 6)
        kb = rng.randint(1 if k < 3 else 2, k)
    return dict(op=op, dims=_txt(dims), block="4,4,4,4", levels=levels, nvec=nvec, nvec2=nvec2, precision=prec,
                nrhs=k, rhs_batch=kb, sap_post=rng.randint(2, 3), restart=rng.choice([4, 6, 10]))


# ---------------------------------------------------------------------------
# inputs

def _ints(s):
    return tuple(int(x) for x in s.split(","))


def _vol(case):
    d = _ints(case["dims"])
    return d[0] * d[1] * d[2] * d[3]


def _mm(a, b):
    return a[..., :, 0:1] * b[..., 0:1, :] + a[..., :, 1:2] * b[..., 1:2, :] + a[..., :, 2:3] * b[..., 2:3, :]


def _links(dims, seed):
    """U = exp(i eps H), H = sum_a h_a lambda_a / 2, h_a ~ N(0,1)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    gm = torch.from_numpy(synth._GM).to("cuda") * (0.5j * EPS)
    h = torch.randn(tuple(dims) + (4, 8), generator=gen, device="cuda", dtype=torch.float64)
    A = torch.zeros(tuple(dims) + (4, 3, 3), device="cuda", dtype=torch.complex128)
    for a in range(8):
        A += h[..., a, None, None] * gm[a]
    # |A| stays below 4: exp(A) = exp(A/8)^8, 12 terms of the series
    A *= 0.125
    eye = torch.eye(3, device="cuda", dtype=torch.complex128)
    E = eye + A / 12.0
    for k in range(11, 0, -1):
        E = eye + _mm(A, E) / k
    for _ in range(3):
        E = _mm(E, E)
    return E.contiguous()


def _gauss(shape, seed, dtype="complex128"):
    return synth.gaussian_device(shape, seed, dtype=dtype)


def _seed(seed, k):
    return (int(seed) * 1000003 + 7919 * k) % (1 << 62)


def _params(case):
    blocks = [_ints(case["block"])]
    nvec = [case["nvec"]]
    if case["levels"] == 3:
        blocks.append((2, 2, 2, 2))
        nvec.append(case["nvec2"])
    return ddamg.default_params(levels=case["levels"], block=blocks, nvec=nvec, precision=case["precision"],
                                setup_iters=1, coarse_setup_iters=1, coarse_mu_factor=DELTA,
                                sap_post=case["sap_post"], restart=case["restart"], rhs_batch=case["rhs_batch"])


def _init_vectors(case, seed):
    dims = _ints(case["dims"])
    dt = "complex128" if case["precision"] == "fp64" else "complex64"
    vecs = [_gauss((case["nvec"],) + dims + (4, 3), _seed(seed, 3), dt)]
    if case["levels"] == 3:
        cd = tuple(d // b for d, b in zip(dims, _ints(case["block"])))
        vecs.append(_gauss((case["nvec2"],) + cd + (2 * case["nvec"],), _seed(seed, 4)))
    return vecs


def _net_params(case, seed):
    """Weights of the given shapes with gates that are in use."""
    rng = np.random.default_rng(_seed(seed, 5))
    W, a, b = synth.net_init_weights(case["chan"], case["layers"], _seed(seed, 6))
    a = [0.02 * rng.standard_normal(len(v)) for v in a]
    b = [0.2 * rng.standard_normal(len(v)) for v in b]
    return W, a, b


def _net_target(case, seed):
    """Orthonormal fields per aggregate half (what a plain setup's P holds)."""
    dims, blk, C = _ints(case["dims"]), _ints(case["block"]), case["chan"]
    g = _gauss((C,) + dims + (4, 3), _seed(seed, 7))
    m = _to_aggregates(g, dims, blk).cpu()
    q = torch.linalg.qr(m)[0].to("cuda")
    return _from_aggregates(q, dims, blk, C).contiguous()


def _to_aggregates(f, dims, blk):
    """[C, T,Z,Y,X, 4, 3] -> [blocks, 2, rows, C]"""
    C = f.shape[0]
    nb = [d // b for d, b in zip(dims, blk)]
    s = f.reshape(C, nb[0], blk[0], nb[1], blk[1], nb[2], blk[2], nb[3], blk[3], 2, 6)
    s = s.permute(1, 3, 5, 7, 9, 2, 4, 6, 8, 10, 0)
    return s.reshape(nb[0] * nb[1] * nb[2] * nb[3], 2, blk[0] * blk[1] * blk[2] * blk[3] * 6, C)


def _from_aggregates(m, dims, blk, C):
    nb = [d // b for d, b in zip(dims, blk)]
    s = m.reshape(nb[0], nb[1], nb[2], nb[3], 2, blk[0], blk[1], blk[2], blk[3], 6, C)
    s = s.permute(10, 0, 5, 1, 6, 2, 7, 3, 8, 4, 9)
    return s.reshape((C,) + tuple(dims) + (4, 3))


def _context(case):
    return ddamg.DDAMG(_ints(case["dims"]), _ints(case["block"]), KAPPA, CSW, MU,
                       stream=torch.cuda.current_stream().cuda_stream)


def prepare(case, seed):
    op, dims = case["op"], _ints(case["dims"])
    mg = _context(case)
    U = _links(dims, _seed(seed, 1))
    s = dict(case=case, mg=mg)
    if op == "field":
        s["U"] = U
        s["psi"] = _gauss(dims + (4, 3), _seed(seed, 2))
        return s
    mg.set_gauge(U)
    mg._keep = None
    del U
    if op in ("dirac", "dirac_noalloc"):
        s["psi"] = _gauss(dims + (4, 3), _seed(seed, 2))
        if op == "dirac_noalloc":
            s["out"] = torch.empty_like(s["psi"])
    elif op in ("dirac_multi", "sap"):
        s["psi"] = _gauss((case["nfields"],) + dims + (4, 3), _seed(seed, 2))
    elif op in ("solve", "setup_solve"):
        s["b"] = _gauss((case["nrhs"],) + dims + (4, 3), _seed(seed, 2))
        s["params"] = _params(case)
        s["vecs"] = _init_vectors(case, seed)
        if op == "solve":
            mg.setup(s["params"], s.pop("vecs"))
    else:
        W, a, b = _net_params(case, seed)
        mg.net_create(case["layers"], case["chan"])
        mg.net_set_params(ddamg.pack_net(W, a, b))
        s["psi"] = _gauss((case["chan"],) + dims + (4, 3), _seed(seed, 2))
        if op == "net_grad":
            s["target"] = _net_target(case, seed)
    torch.cuda.empty_cache()
    return s


def _sap_device(mg, b, x, iters, mr_steps, precision):
    """ddamg_sap_multi of the C interface on fields that live on the device
    (x updated in place)."""
    mg._check(ddamg._lib.ddamg_sap_multi(mg._h, int(b.shape[0]), ctypes.c_void_p(b.data_ptr()),
                                         ctypes.c_void_p(x.data_ptr()), int(iters), int(mr_steps),
                                         ddamg.PRECISIONS[precision], 1))


def run(state):
    case, mg = state["case"], state["mg"]
    op = case["op"]
    if op in ("dirac", "dirac_multi"):
        f = mg.apply_dirac if op == "dirac" else mg.apply_dirac_multi
        y = f(state["psi"], precision=case["precision"])
        return y if case["precision"] == "fp64" else y.to(torch.complex64)
    if op == "dirac_noalloc":
        return mg.apply_dirac_noalloc(state["psi"], state["out"])
    if op == "sap":
        x = torch.zeros_like(state["psi"])
        _sap_device(mg, state["psi"], x, case["iters"], case["mr_steps"], case["precision"])
        return x if case["precision"] == "fp64" else x.to(torch.complex64)
    if op == "field":
        mg.set_gauge(state["U"])
        return mg.apply_dirac(state["psi"])
    if op == "solve":
        return mg.solve(state["b"], tol=TOL)[0]
    if op == "setup_solve":
        mg.setup(state["params"], state["vecs"])
        return mg.solve(state["b"], tol=TOL)[0]
    if op == "net_forward":
        return mg.net_forward(state["psi"]).to(torch.complex64)
    loss, g = mg.net_loss_grad(state["psi"], state["target"])
    return {"loss": np.float32(loss), "grad": g.astype(np.float32)}


# ---------------------------------------------------------------------------
# what a pass cannot do without.  Per site: links 36 complex, clover 72 reals,
# odd-site inverse factors 36 reals (half of the sites); D(mu) 2184 flops (eight
# hops 1632, the site term 552); one SAP iteration (4932 + 2604 n_MR) flops per
# field.  A solve counts the iterations such solves take (20 outer ones, each
# one D(mu) and the fine smoother's iterations); the coarse levels come on top.

_OPB = {"fp64": 576 + 576, "fp32": 288 + 288, "fp16": 144 + 288, "bf16": 144 + 288}


def work(case):
    V, op = _vol(case), case["op"]
    if op in ("dirac", "dirac_noalloc", "dirac_multi"):
        k = case.get("nfields", 1)
        io = 384 if case["precision"] == "fp64" else 192 + 96
        return dict(bytes=float(V) * (_OPB[case["precision"]] + k * io), flops=2184.0 * V * k)
    if op == "sap":
        k, p = case["nfields"], case["precision"]
        io = 384 if p == "fp64" else 192 + 96
        return dict(bytes=float(V) * (_OPB[p] + (288 if p == "fp64" else 144) + k * io),
                    flops=float(V) * k * case["iters"] * (4932 + 2604 * case["mr_steps"]))
    if op == "field":
        # six planes of four leaves, three 3x3 products each (198 flops)
        return dict(bytes=float(V) * (576 + 384), flops=float(V) * (6 * 4 * 3 * 198 + 2184))
    if op in ("solve", "setup_solve"):
        k = case["nrhs"]
        it = 20.0 * (2184 + case["sap_post"] * (4932 + 2604 * 4))
        if op == "setup_solve":  # initial smoothing and one iteration of every test vector
            it_setup = case["nvec"] * (3 + case["sap_post"]) * (4932 + 2604.0 * 4)
            vec = case["nvec"] * (192 if case["precision"] == "fp64" else 96)
        else:
            it_setup, vec = 0.0, 0
        return dict(bytes=float(V) * (576 + 576 + vec + k * 384), flops=float(V) * (k * it + it_setup))
    L, C = case["layers"], case["chan"]
    f = 8.0 * 9 * C * C * 16 * 3 * L * V
    if op == "net_forward":
        return dict(bytes=float(V) * (576 + C * (192 + 96)), flops=f)
    return dict(bytes=float(V) * (576 + C * 384) + 16.0 * L * 9 * C * C * 16, flops=3 * f)


# ---------------------------------------------------------------------------
# the same in 64 bits, by plain torch.  Gamma matrices of the chiral basis, one
# nonzero entry per row: (gamma_mu psi)_s = phase[mu][s] psi_{perm[mu][s]}

_PERM = [(2, 3, 0, 1), (2, 3, 0, 1), (3, 2, 1, 0), (3, 2, 1, 0)]
_PHASE = [(-1, -1, -1, -1), (-1j, 1j, 1j, -1j), (-1, 1, 1, -1), (-1j, -1j, 1j, 1j)]  # T Z Y X


def _gamma(mu):
    g = torch.zeros(4, 4, dtype=torch.complex128)
    for s in range(4):
        g[s, _PERM[mu][s]] = _PHASE[mu][s]
    return g


def _dag(m):
    return m.mH.resolve_conj()


def _clover(U):
    """The two chirality blocks [.., 2, 6, 6] of (m0 + 4) + A."""
    dims = U.shape[:4]
    sh = lambda f, mu, s: torch.roll(f, -s, dims=mu)  # noqa: E731  f(x + s mu)
    A = torch.zeros(tuple(dims) + (2, 2, 3, 2, 3), dtype=torch.complex128, device=U.device)
    for mu in range(4):
        for nu in range(mu + 1, 4):
            a, b = U[..., mu, :, :], U[..., nu, :, :]
            am, bm, an, bn = sh(a, mu, -1), sh(b, mu, -1), sh(a, nu, -1), sh(b, nu, -1)
            q = _mm(_mm(a, sh(b, mu, 1)), _mm(_dag(sh(a, nu, 1)), _dag(b)))
            q += _mm(_mm(b, _dag(sh(am, nu, 1))), _mm(_dag(bm), am))
            q += _mm(_mm(_dag(am), _dag(sh(bm, nu, -1))), _mm(sh(am, nu, -1), bn))
            q += _mm(_mm(_dag(bn), an), _mm(sh(bn, mu, 1), _dag(a)))
            F = (q - _dag(q)) / 8.0
            s = 0.5j * (_gamma(mu) @ _gamma(nu) - _gamma(nu) @ _gamma(mu)) * (0.5j * CSW)
            for c in range(2):
                for i in range(2):
                    for j in range(2):
                        v = complex(s[2 * c + i, 2 * c + j])
                        if v != 0:
                            A[..., c, i, :, j, :] += v * F
    A = A.reshape(tuple(dims) + (2, 6, 6))
    A += (1.0 / (2.0 * KAPPA)) * torch.eye(6, dtype=torch.complex128, device=U.device)
    return A


def _site(H, psi):
    """((m0 + 4) + A + i mu gamma5) psi, psi [K, T,Z,Y,X, 4, 3]"""
    p = psi.reshape(psi.shape[:-2] + (2, 6))
    out = torch.zeros_like(p)
    for j in range(6):
        out += H[..., j] * p[..., j:j + 1]
    tw = torch.tensor([-1j * MU, 1j * MU], dtype=torch.complex128, device=psi.device)
    return (out + tw[:, None] * p).reshape(psi.shape)


def _hop(U, psi):
    """-1/2 sum of the eight hops of psi [K, T,Z,Y,X, 4, 3]"""
    out = torch.zeros_like(psi)
    for mu in range(4):
        u = U[..., mu, :, :]
        ph = torch.tensor(_PHASE[mu], dtype=torch.complex128, device=psi.device)[:, None]
        for sign in (1, -1):
            if sign > 0:
                f, m = torch.roll(psi, -1, dims=1 + mu), u
            else:
                f, m = torch.roll(psi, 1, dims=1 + mu), _dag(torch.roll(u, 1, dims=mu))
            w = m[..., None, :, 0] * f[..., 0:1] + m[..., None, :, 1] * f[..., 1:2] + m[..., None, :, 2] * f[..., 2:3]
            out -= 0.5 * w
            out += (0.5 * sign) * ph * w[..., list(_PERM[mu]), :]
    return out


def _stored(U, precision):
    """The links as the precision option stores them (rounded to nearest even)."""
    if precision not in ("fp16", "bf16"):
        return U
    t = torch.float16 if precision == "fp16" else torch.bfloat16
    r = torch.view_as_real(U)
    return torch.view_as_complex(r.to(torch.float32).to(t).to(torch.float64))


def _inverse6(M):
    """Inverse of [.., 6, 6] by elimination (the blocks are diagonally dominant)."""
    n = 6
    a = torch.cat([M, torch.eye(n, dtype=M.dtype, device=M.device).expand(M.shape)], dim=-1).clone()
    for k in range(n):
        a[..., k, :] /= a[..., k, k].clone()[..., None]
        for i in range(n):
            if i != k:
                a[..., i, :] -= a[..., i, k].clone()[..., None] * a[..., k, :]
    return a[..., n:].contiguous()


def _sap_exact(case, U, H, b):
    dims, blk = _ints(case["dims"]), _ints(case["block"])
    nb = [d // c for d, c in zip(dims, blk)]
    dev = b.device
    g = torch.meshgrid(*[torch.arange(d, device=dev) for d in dims], indexing="ij")
    par = (g[0] + g[1] + g[2] + g[3]) % 2
    col = (g[0] // blk[0] + g[1] // blk[1] + g[2] // blk[2] + g[3] // blk[3]) % 2
    tw = torch.tensor([-1j * MU, 1j * MU], dtype=torch.complex128, device=dev)
    Tinv = _inverse6(H + tw[:, None, None] * torch.eye(6, dtype=torch.complex128, device=dev))

    def site_inv(v):
        p = v.reshape(v.shape[:-2] + (2, 6))
        out = torch.zeros_like(p)
        for j in range(6):
            out += Tinv[..., j] * p[..., j:j + 1]
        return out.reshape(v.shape)

    def block_sum(v):  # [K, T,Z,Y,X] -> the sum of the site's block at every site
        K = v.shape[0]
        s = v.reshape(K, nb[0], blk[0], nb[1], blk[1], nb[2], blk[2], nb[3], blk[3]).sum(dim=(2, 4, 6, 8), keepdim=True)
        return s.expand(K, nb[0], blk[0], nb[1], blk[1], nb[2], blk[2], nb[3], blk[3]).reshape(v.shape)

    x = torch.zeros_like(b)
    for _ in range(case["iters"]):
        for c in (0, 1):
            r = b - _site(H, x) - _hop(U, x)
            E = ((col == c) & (par == 0))[..., None, None].to(torch.float64)
            O = ((col == c) & (par == 1))[..., None, None].to(torch.float64)
            rho = E * r - E * _hop(U, O * site_inv(O * r))
            e = torch.zeros_like(b)
            for _ in range(case["mr_steps"]):
                q = E * (_site(H, rho) - _hop(U, O * site_inv(O * _hop(U, rho))))
                qr = block_sum((q.conj() * rho).sum(dim=(-1, -2)))
                qq = block_sum((q.real ** 2 + q.imag ** 2).sum(dim=(-1, -2)))
                al = torch.where(qq > 0, qr / torch.where(qq > 0, qq, torch.ones_like(qq)), torch.zeros_like(qr))
                e = e + al[..., None, None] * rho
                rho = rho - al[..., None, None] * q
            x = x + e + O * site_inv(O * (r - _hop(U, e)))
    return x


def _solve_exact(U, H, b):
    """Conjugate gradients on gamma5 D(-mu) gamma5 D(mu) x = ..., per source."""
    g5 = torch.tensor([-1.0, -1.0, 1.0, 1.0], device=b.device, dtype=torch.float64)[:, None]
    tw = torch.tensor([-2j * MU, 2j * MU], dtype=torch.complex128, device=b.device)

    def D(v):
        return _site(H, v) + _hop(U, v)

    def Ddag(v):  # gamma5 D(-mu) gamma5
        w = g5 * v
        y = D(w) - (tw[:, None] * w.reshape(w.shape[:-2] + (2, 6))).reshape(w.shape)
        return g5 * y

    def dot(a, c):
        return (a.conj() * c).real.flatten(1).sum(1)

    x = torch.zeros_like(b)
    ex = (slice(None),) + (None,) * (b.ndim - 1)
    for _ in range(3):  # restarts from the true residual
        r = Ddag(b - D(x))
        p, rr = r.clone(), dot(r, r)
        r0 = rr.clone()
        for k in range(4000):
            q = D(p)
            al = rr / dot(q, q)
            x = x + al[ex] * p
            r = r - al[ex] * Ddag(q)
            rn = dot(r, r)
            if k % 25 == 24 and bool((rn < 1e-26 * r0).all()):
                break
            p = r + (rn / rr)[ex] * p
            rr = rn
    return x


def _net_apply(U, case, x, W, a, b):
    C, dims = case["chan"], _ints(case["dims"])
    V = _vol(case)
    for l in range(case["layers"]):
        tx = [x]
        for sign in (1, -1):
            for mu in range(4):
                u = U[..., mu, :, :]
                if sign > 0:
                    f, m = torch.roll(x, -1, dims=1 + mu), u
                else:
                    f, m = torch.roll(x, 1, dims=1 + mu), _dag(torch.roll(u, 1, dims=mu))
                tx.append(m[..., None, :, 0] * f[..., 0:1] + m[..., None, :, 1] * f[..., 1:2]
                          + m[..., None, :, 2] * f[..., 2:3])
        X = torch.stack(tx).reshape(9, C, V, 4, 3).permute(0, 1, 3, 2, 4).reshape(9 * C * 4, V * 3)
        M = W[l].permute(1, 3, 0, 2, 4).reshape(C * 4, 9 * C * 4)
        z = (M @ X).reshape(C, 4, V, 3).permute(0, 2, 1, 3).reshape((C,) + dims + (4, 3))
        if l < case["layers"] - 1:
            n = (z.real ** 2 + z.imag ** 2).sum(dim=(-1, -2))
            ex = (slice(None), None, None, None, None)
            z = z * torch.sigmoid(a[l][ex] * n + b[l][ex])[..., None, None]
        x = z
    return x


def _net_exact(case, seed, U):
    dims, blk = _ints(case["dims"]), _ints(case["block"])
    W, a, b = _net_params(case, seed)
    grad = case["op"] == "net_grad"
    W = [torch.from_numpy(np.ascontiguousarray(w)).to("cuda").requires_grad_(grad) for w in W]
    a = [torch.from_numpy(v).to("cuda").requires_grad_(grad) for v in a]
    b = [torch.from_numpy(v).to("cuda").requires_grad_(grad) for v in b]
    x = _gauss((case["chan"],) + dims + (4, 3), _seed(seed, 2))
    y = _net_apply(U, case, x, W, a, b)
    if not grad:
        return y
    Y = _to_aggregates(y, dims, blk)
    Q = _to_aggregates(_net_target(case, seed), dims, blk)
    B, rows, C = Y.shape[0] * 2, Y.shape[2], case["chan"]
    Y, Q = Y.reshape(B, rows, C).cpu(), Q.reshape(B, rows, C).cpu()
    G, P = Y.mH @ Y, Y.mH @ Q
    R = Q - Y @ torch.linalg.solve(G, P)
    loss = (R.real ** 2 + R.imag ** 2).sum() / (Q.real ** 2 + Q.imag ** 2).sum()
    loss.backward()
    parts = [torch.view_as_real(w.grad.resolve_conj()).reshape(-1) for w in W]
    for p, q in zip(a, b):
        parts += [p.grad.reshape(-1), q.grad.reshape(-1)]
    return {"loss": float(loss), "grad": torch.cat(parts)}


def exact(case, seed):
    op, dims = case["op"], _ints(case["dims"])
    if op == "setup_solve" or (op == "solve" and _vol(case) * case["nrhs"] > 70000):
        return None  # conjugate gradients would take too long
    with torch.no_grad():
        U = _links(dims, _seed(seed, 1))
    if op.startswith("net"):
        return _net_exact(case, seed, U)
    with torch.no_grad():
        H = _clover(U)
        U = _stored(U, case.get("precision", "fp64")) if op != "solve" else U
        if op in ("dirac", "dirac_noalloc", "field"):
            psi = _gauss(dims + (4, 3), _seed(seed, 2))[None]
            return (_site(H, psi) + _hop(U, psi))[0]
        if op == "dirac_multi":
            K = case["nfields"]
            psi = _gauss((K,) + dims + (4, 3), _seed(seed, 2))
            return torch.cat([_site(H, psi[k:k + 1]) + _hop(U, psi[k:k + 1]) for k in range(K)])
        if op == "sap":
            psi = _gauss((case["nfields"],) + dims + (4, 3), _seed(seed, 2))
            return torch.cat([_sap_exact(case, U, H, psi[k:k + 1]) for k in range(case["nfields"])])
        return _solve_exact(U, H, _gauss((case["nrhs"],) + dims + (4, 3), _seed(seed, 2)))
