"""Batches on layers of few neurons, whose gate segments are of at most 32 rows (64 for 2..4 tokens), and at
the d_ff where that ends, against the oracle."""
import pytest

from paper_2609_31975_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from tests import gpu_util
    return gpu_util


@pytest.mark.parametrize("dense", [False, True], ids=["sparse", "dense"])
@pytest.mark.parametrize("d_ff", [1, 31, 33, 65, 4096, 4097, 8192, 8193])
@pytest.mark.parametrize("T,r,wdt", [(3, 0, wl.BF16), (5, 16, wl.BF16), (16, 0, wl.I8), (20, 8, wl.F32), (64, 0, wl.BF16)])
def test_segments(gu, T, r, wdt, d_ff, dense):
    d, t = 48, 1.3
    inp = wl.make_inputs(701, T, d, d_ff, r=r, wdt=wdt)
    y, idx, act, _ = (gu.run_gpu_q if wdt == wl.I8 else gu.run_gpu)(gu.DevInputs(inp), t, dense=dense)
    res = gu.run_oracle(inp, t, dense=dense)
    big = d_ff >= 4096  # y of a few neurons is rebuilt from the kernel's activations instead
    gu.check_parity(res, y, idx, act, t, wl.BF16 if wdt != wl.F32 else wdt, dense=dense, what=f"T={T} d_ff={d_ff}",
                    check_y=big)
    if not big:
        gu.check_rebuilt(inp, y, idx, act, wdt, what=f"T={T} d_ff={d_ff}")
