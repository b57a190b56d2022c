"""Which of its two forms a fine smoother sweep takes (one thread or two to a
pair of slots), on the GPU: both forms give the same field at the edges of the
rule, and the rule costs no time where wavefronts are mostly empty.

Bars, fixed before the first run: each form is within 1e-5 of the exact sweep
(the FP32 SAP bar of the parity tests), so 2e-5 apart.  Times: a field of
small blocks alone against two in one call, 0.53 of their time in the form for
one thread a pair and 0.83 in the other, so at most 0.68; fewer blocks against
more in FP16, 0.88 and 1.19 of their time, so at most 1.03."""
import ctypes
import time

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
    from paper_1611_01034_amd import synth
    ctx = dd.DDAMG(dims, block, KAPPA, CSW, MU, stream=torch.cuda.current_stream().cuda_stream)
    ctx.set_gauge(synth.gauge_field_device(dims, 0.3, 9601))
    return ctx


def _sap(dd, ctx, b, x, iters, prec):
    ctx._check(dd._lib.ddamg_sap_multi(ctx._h, int(b.shape[0]), ctypes.c_void_p(b.data_ptr()),
                                       ctypes.c_void_p(x.data_ptr()), iters, 3, dd.PRECISIONS[prec], 1))


@pytest.mark.parametrize("dims,block,precs", [
    ((12, 12, 12, 12), (2, 2, 2, 2), ("fp32", "fp16", "bf16")),   # 8 pairs: 648 workgroups, 1296 wavefronts
    ((16, 16, 16, 8), (2, 2, 2, 2), ("fp32", "bf16")),            # 1024: 2048, the last that take two threads
    ((16, 12, 12, 12), (2, 2, 2, 2), ("fp16",)),                  # 864: 1728, 3456 for two fields
    ((24, 12, 12, 12), (2, 2, 2, 2), ("fp16",)),                  # 1296: 2592
    ((24, 24, 16, 12), (4, 4, 4, 2), ("fp32",)),                  # 64 pairs: 432 workgroups, 864
    ((24, 24, 24, 16), (4, 4, 4, 2), ("fp32",)),                  # 64 pairs: 864, 1728
    ((36, 32, 24, 24), (6, 4, 2, 2), ("fp32",)),                  # 48 pairs: 3456, 6912
    ((24, 24, 24, 20), (6, 2, 2, 2), ("fp32",))])                 # 24 pairs: 2880, 5760
def test_both_forms_agree(dd, dims, block, precs):
    from paper_1611_01034_amd import synth
    with _ctx(dd, dims, block) as ctx:
        b = synth.gaussian_device((2,) + dims + (4, 3), 9602)
        x0 = synth.gaussian_device((2,) + dims + (4, 3), 9603)
        for prec in precs:
            print(f"sap forms: {dims} {block} {prec}", flush=True)
            many = x0.clone()
            _sap(dd, ctx, b, many, 2, prec)
            for k in range(2):
                one = x0[k:k + 1].clone()
                _sap(dd, ctx, b[k:k + 1], one, 2, prec)
                d = torch.linalg.vector_norm(one[0] - many[k]) / torch.linalg.vector_norm(many[k])
                assert float(d) <= 2e-5, (prec, k, float(d))


def _seconds(dd, ctx, b, iters, prec):
    x = torch.zeros_like(b)
    best = float("inf")
    for _ in range(8):
        torch.cuda.synchronize()
        t = time.perf_counter()
        _sap(dd, ctx, b, x, iters, prec)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


def test_one_field_of_small_blocks_costs_its_share(dd):
    from paper_1611_01034_amd import synth
    dims = (28, 28, 24, 24)
    with _ctx(dd, dims, (2, 2, 2, 2)) as ctx:
        b = synth.gaussian_device((2,) + dims + (4, 3), 9604)
        print("one FP32 field of 16-site blocks", flush=True)
        one, two = _seconds(dd, ctx, b[:1], 6, "fp32"), _seconds(dd, ctx, b, 6, "fp32")
        assert one <= 0.68 * two, (one, two)


def test_fewer_small_blocks_take_no_longer(dd):
    from paper_1611_01034_amd import synth
    t = []
    for dims in ((16, 16, 12, 12), (16, 16, 16, 16)):
        with _ctx(dd, dims, (2, 2, 2, 2)) as ctx:
            print(f"FP16 sweep of 16-site blocks: {dims}", flush=True)
            t.append(_seconds(dd, ctx, synth.gaussian_device((1,) + dims + (4, 3), 9605), 40, "fp16"))
    assert t[0] <= 1.03 * t[1], t
