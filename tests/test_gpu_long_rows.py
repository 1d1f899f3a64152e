"""Single-token LoPA calls on rows of more than 8 chunks a lane, at both sides of the rank rule that says
whether x for the W_up dots waits in LDS, against the oracle."""
import pytest

from paper_2609_31975_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from tests import gpu_util
    return gpu_util


@pytest.mark.parametrize("full", [False, True], ids=["default", "full"])
@pytest.mark.parametrize("d,r,wdt", [(4104, 512, wl.BF16), (4104, 520, wl.BF16), (6400, 720, wl.BF16), (6408, 720, wl.BF16),
                                     (4104, 728, wl.BF16), (4104, 4104, wl.BF16), (2052, 512, wl.F32), (2052, 516, wl.F32),
                                     (4096, 700, wl.F32), (2052, 2052, wl.F32)])
def test_long_rows(gu, d, r, wdt, full):
    d_ff, t = 333, 0.8
    inp = wl.make_inputs(801, 1, d, d_ff, r=r, wdt=wdt)
    dev = gu.DevInputs(inp)
    form = gu.Form(act=1, silu_up=True, form=wl.make_form(801, d, d_ff, r), use_g=True, rms_norm=True,
                   use_gain=True) if full else None
    y, idx, act, _ = gu.run_gpu_ex(dev, t, form) if full else gu.run_gpu(dev, t)
    res = gu.run_oracle(inp, t, form=form)
    gu.check_parity(res, y, idx, act, t, wdt, what=f"d={d} r={r}", act_value=form.act_value if full else None)
