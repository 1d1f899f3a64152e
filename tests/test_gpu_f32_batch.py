"""Batches with fp32 weights on the fp32 matrix-core kernels, against the oracle: edges of token
tiles, of segments, of k steps (16 elements) and of column groups, each gating and form."""
import pytest

from paper_2609_31975_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from tests import gpu_util
    return gpu_util


# T, d, d_ff, r, threshold; widths of 1, 4, 5, 64 + 1 and 256 + 1 chunks of 4
SHAPES = [
    (2, 4, 3, 0, 0.0),            # one chunk, one segment of three rows
    (3, 20, 130, 4, 0.3),         # a k step of one chunk, a rank of one chunk
    (4, 260, 1000, 36, 1.0),
    (16, 1028, 999, 60, 1.2),     # one full token tile, an odd d_ff
    (17, 260, 700, 0, 1.0),       # packed tokens, one token in the second tile
    (33, 132, 520, 20, 1.2),      # four token tiles, the third with one token
    (64, 1028, 1100, 0, 1.4),     # the largest pass
    (65, 64, 300, 8, 1.2),        # two passes, the second of one token (single-token kernels)
    (5, 136, 24600, 24, 1.6),     # two workgroups a CU, ragged segments
    (6, 260, 1000, 38, 1.0),      # a rank of no whole chunk: element-wise kernels
]


@pytest.mark.parametrize("dense", [False, True], ids=["sparse", "dense"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "T%d_d%d_dff%d_r%d" % s[:4])
def test_f32_batch(gu, shape, dense):
    T, d, d_ff, r, t = shape
    inp = wl.make_inputs(501, T, d, d_ff, r=r, wdt=wl.F32)
    y, idx, act, _ = gu.run_gpu(gu.DevInputs(inp), t, dense=dense)
    res = gu.run_oracle(inp, t, dense=dense)
    gu.check_parity(res, y, idx, act, t, wl.F32, dense=dense, what=str(shape))


@pytest.mark.parametrize("T", [4, 20, 50])
def test_f32_batch_full_form(gu, T):
    d, d_ff, r, t = 260, 1000, 36, 1.5
    inp = wl.make_inputs(502, T, d, d_ff, r=r, wdt=wl.F32)
    form = gu.Form(act=1, silu_up=True, form=wl.make_form(502, d, d_ff, r), use_g=True, rms_norm=True, use_gain=True)
    y, idx, act, _ = gu.run_gpu_ex(gu.DevInputs(inp), t, form)
    res = gu.run_oracle(inp, t, form=form)
    gu.check_parity(res, y, idx, act, t, wl.F32, what=f"full form T={T}", act_value=form.act_value)


@pytest.mark.parametrize("T", [17, 80])
@pytest.mark.parametrize("wdt", [wl.F32, wl.BF16], ids=["f32", "bf16"])
def test_nan_tokens_leave_no_z_tag(gu, wdt, T):
    """Tokens that hold the signalling NaN that tags a published z: a batch leaves no such word in the
    workspace, where a later single-token LoPA call of a larger rank would take it for one."""
    import numpy as np
    import torch
    from paper_2609_31975_amd import ffn
    tag, d = 0x7FA5A5A5, 256
    inp = wl.make_inputs(503, T, d, 8, wdt=wdt)
    bits = np.full((T, d), tag, np.uint32)
    if wdt == wl.BF16:
        bits[:, 0::2] = 0xA5A50000  # the low half of a word of two bf16
    inp.x = bits.view(np.float32)
    dev = gu.DevInputs(inp)
    ws = ffn.alloc_workspace(T, d, 8)
    ffn.ffn_sparse_forward(dev.x, dev.w_gate, dev.w_up, dev.w_down_t, 1.0, torch.empty_like(dev.x), ws)
    assert not bool((ws.view(torch.int32) == tag).any())
