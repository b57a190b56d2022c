"""Checks of inputs with 2^32 numbers or more, on the GPU: the library looks at
all of them (a launch holds fewer than 2^32 threads)."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def test_non_finite_link_of_a_large_field():
    """A field of 96 x 96 x 96 x 72 links (4.6e9 reals, 34 GiB) with one NaN is
    refused, wherever it is."""
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 170 << 30:
        pytest.skip("needs 170 GiB of free device memory")
    from paper_1611_01034_amd import ddamg
    dims, block = (96, 96, 96, 72), (4, 4, 4, 4)
    U = torch.zeros(dims + (4, 3, 3), dtype=torch.complex128, device="cuda")
    r = torch.view_as_real(U).reshape(-1)
    assert r.numel() >= 2 ** 32
    status = []
    with ddamg.DDAMG(dims, block, 0.13729, 0.0, 0.1, stream=torch.cuda.current_stream().cuda_stream) as ctx:
        for where in (0, 2 ** 31, 2 ** 32 + 5, -1):
            print(f"NaN at {where} of {r.numel()}", flush=True)
            r[where] = float("nan")
            status.append(ddamg._lib.ddamg_set_gauge(ctx._h, U.data_ptr(), 1))
            r[where] = 0.0
    del U, r
    torch.cuda.empty_cache()
    assert status == [ddamg.NUMERICAL] * 4
