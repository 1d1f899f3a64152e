"""Calls of more than 64 tokens on the wide kernels (bf16, int8, int4 weights), against the oracle:
edges of token tiles and blocks, of segments, of an iteration's 64 elements and of column groups."""
import numpy as np
import pytest

from paper_2609_31975_amd import workloads as wl

pytestmark = pytest.mark.gpu

BF16, I8, I4 = wl.BF16, wl.I8, wl.I4


@pytest.fixture(scope="module")
def gu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a ROCm device"
    from tests import gpu_util
    return gpu_util


# T, d, d_ff, r, wdt, threshold
SHAPES = [
    (65, 8, 3, 0, BF16, 0.0),           # 64 tokens, then one on the single-token kernels
    (66, 72, 130, 8, BF16, 0.3),        # 64 tokens, then two
    (81, 8, 3, 0, BF16, 0.0),           # one chunk, one segment of three rows, a tile of one token
    (97, 72, 130, 8, BF16, 0.3),        # segments of 43 rows, a k step of one chunk, a rank of one
    (65, 264, 2500, 0, BF16, 1.6),      # one token past 64 on the wide kernels
    (65, 2048, 300, 0, I4, 1.6),        # ... and not: long rows of codes, few neurons
    (96, 64, 300, 64, I8, 1.6),         # LoPA with codes on a small layer: 64 tokens, then 32
    (80, 264, 1000, 40, BF16, 1.6),
    (80, 136, 1000, 0, BF16, 3.0),      # small unions, some segments with none
    (100, 1032, 999, 72, BF16, 1.6),    # an odd d_ff; 129 chunks a row; nine column groups
    (128, 264, 2100, 0, BF16, 1.0),     # one full block
    (129, 264, 12300, 40, BF16, 2.2),   # two blocks, segments of 128 and 127 rows, unions past 64
    (129, 136, 12300, 0, BF16, -9.0),   # everything active
    (200, 136, 12289, 16, BF16, 3.1),   # segments of up to 128 rows with unions of at most 64
    (300, 264, 1000, 40, BF16, 1.6),    # several passes
    (193, 72, 700, 0, BF16, 1.6),       # several passes, the last one small
    (100, 272, 999, 48, I8, 1.6),
    (130, 528, 12300, 0, I8, 2.4),
    (100, 288, 999, 64, I4, 1.6),
    (130, 544, 12300, 0, I4, 2.4),
]


@pytest.mark.parametrize("dense", [False, True], ids=["sparse", "dense"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "T%d_d%d_dff%d_r%d_w%d" % s[:5])
def test_wide(gu, shape, dense):
    T, d, d_ff, r, wdt, t = shape
    inp = wl.make_inputs(601, T, d, d_ff, r=r, wdt=wdt)
    dev = gu.DevInputs(inp)
    y = (gu.run_gpu_q if wdt in (I8, I4) else gu.run_gpu)(dev, t, dense=dense)[0]
    res = gu.run_oracle(inp, t, dense=dense)
    gu.check_parity(res, y, None, None, t, BF16, dense=dense, what=str(shape))
    # the tolerance of bf16 weights is wide: the tokens' two bf16 parts hold 2^-16 of an element
    assert gu.rel_err(y, res.y) <= 3e-5


# 33..64 tokens, rows shorter than the wide kernels take (the register-tiled ones run them)
@pytest.mark.parametrize("dense", [False, True], ids=["sparse", "dense"])
@pytest.mark.parametrize("shape", [(33, 72, 13957, 24, BF16, 1.6), (64, 136, 16384, 0, BF16, 2.0),
                                   (49, 72, 28650, 40, BF16, 1.8), (64, 80, 14000, 16, I8, 1.6),
                                   (50, 96, 14000, 0, I4, 1.6), (40, 16, 14000, 2048, BF16, 1.6)],
                         ids=lambda s: "T%d_d%d_dff%d_r%d_w%d" % s[:5])
def test_wide_33_to_64(gu, shape, dense):
    T, d, d_ff, r, wdt, t = shape
    inp = wl.make_inputs(605, T, d, d_ff, r=r, wdt=wdt)
    y, idx, act, _ = (gu.run_gpu_q if wdt in (I8, I4) else gu.run_gpu)(gu.DevInputs(inp), t, dense=dense)
    res = gu.run_oracle(inp, t, dense=dense)
    gu.check_parity(res, y, idx, act, t, BF16, dense=dense, what=str(shape))
    assert gu.rel_err(y, res.y) <= 3e-5


def wide64_nseg(ws, T, d, d_ff, r):
    """Segments of 64 rows, in which the wide kernels cut d_ff at 33..64 tokens (the register-tiled ones
    take a whole number of rounds of 256 there)."""
    from paper_2609_31975_amd import ffn
    assert int(ffn.ffn_workspace_active(ws, T, d, d_ff, r)[0][0]) == (d_ff + 63) // 64


# T, d, d_ff, r, weights, threshold, full form, dense: 224 segments of 64 and of 63 .. 64 rows, 448; the
# shortest rows the path takes; tokens of three and four tiles, one in the last
WIDE64 = [
    (33, 2304, 14300, 0, BF16, 1.6, False, False),
    (64, 2304, 14336, 288, BF16, 1.3, True, False),
    (49, 2304, 28650, 40, BF16, 2.2, False, False),
    (33, 2304, 14336, 2304, BF16, 1.6, False, True),
    (64, 2048, 14300, 272, I8, 1.6, True, False),
    (41, 2064, 14336, 0, I8, 2.4, False, False),
    (64, 2048, 14336, 96, I4, 1.6, False, False),
    (50, 2080, 14290, 0, I4, 2.0, True, True),
]


@pytest.mark.parametrize("shape", WIDE64, ids=lambda s: "T%d_d%d_dff%d_r%d_w%d_full%d_dense%d" % (*s[:5], *s[6:]))
def test_wide_kernels_33_to_64(gu, shape):
    """The oracle takes a few of the tokens; every token's active set is checked by its list."""
    T, d, d_ff, r, wdt, t, full, dense = shape
    inp = wl.make_inputs(607, T, d, d_ff, r=r, wdt=wdt)
    lopa = dict(form=wl.make_form(607, d, d_ff, r), use_g=True, rms_norm=True, use_gain=True) if r else {}
    form = gu.Form(act=1, silu_up=True, **lopa) if full else None
    dev = gu.DevInputs(inp)
    if wdt in (I8, I4):
        y, idx, act, ws = gu.run_gpu_q(dev, t, dense=dense, form=form)
    elif full:
        y, idx, act, ws = gu.run_gpu_ex(dev, t, form, dense=dense)
    else:
        y, idx, act, ws = gu.run_gpu(dev, t, dense=dense)
    wide64_nseg(ws, T, d, d_ff, r)
    assert np.all(np.diff(idx) > 0) and (len(idx) == d_ff if dense else (act > 0).any(0).all())
    sel = [0, 15, 16, T // 2, T - 1]
    res = gu.run_oracle(inp, t, dense=dense, x=inp.x[sel], form=form)
    gu.check_parity(res, y[sel], None, None, t, BF16, dense=dense, what=str(shape))
    assert gu.rel_err(y[sel], res.y) <= 3e-5
    for k, tau in enumerate(sel):
        on = np.zeros(d_ff, bool)
        on[idx] = act[tau] > 0
        band = np.abs(res.h[k] - np.float64(np.float32(t))) < gu.BAND
        assert np.array_equal(on[~band], res.active[k][~band]), tau


@pytest.mark.parametrize("wdt", [BF16, I8], ids=["bf16", "i8"])
@pytest.mark.parametrize("r", [0, 48], ids=["std", "lopa"])
def test_wide_full_form(gu, wdt, r):
    T, d, d_ff, t = 150, 272, 1500, 2.0
    inp = wl.make_inputs(602, T, d, d_ff, r=r, wdt=wdt)
    lopa = dict(form=wl.make_form(602, d, d_ff, r), use_g=True, rms_norm=True, use_gain=True) if r else {}
    form = gu.Form(act=1, silu_up=True, **lopa)
    dev = gu.DevInputs(inp)
    y = gu.run_gpu_q(dev, t, form=form)[0] if wdt == I8 else gu.run_gpu_ex(dev, t, form)[0]
    res = gu.run_oracle(inp, t, form=form)
    gu.check_parity(res, y, None, None, t, BF16, what=f"full form w{wdt} r={r}")
    assert gu.rel_err(y, res.y) <= 3e-5


def test_wide_between_other_calls(gu):
    """One workspace, no refill: single-token LoPA calls (whose z slots live in it) around wide ones."""
    import torch
    from paper_2609_31975_amd import ffn
    d, d_ff, r, t, T = 264, 1000, 40, 1.2, 177
    inp = wl.make_inputs(603, T, d, d_ff, r=r, wdt=BF16)
    dev = gu.DevInputs(inp)
    ws = ffn.alloc_workspace(T, d, d_ff, r)
    res = gu.run_oracle(inp, t)
    for n in (1, T, 1, 3, T, 1):
        y = torch.full((n, d), float("nan"), device="cuda")
        ffn.ffn_lopa_sparse_forward(dev.x[:n].contiguous(), dev.lopa_a, dev.lopa_b, dev.w_up, dev.w_down_t, t, y, ws)
        assert gu.rel_err(y.cpu().numpy(), res.y[:n]) <= 3e-5, n


def test_wide_without_a_workspace_argument(gu):
    import torch
    from paper_2609_31975_amd import ffn
    d, d_ff, t, T = 264, 1000, 1.2, 100
    inp = wl.make_inputs(604, T, d, d_ff, wdt=BF16)
    dev = gu.DevInputs(inp)
    y = torch.full((T, d), float("nan"), device="cuda")
    ffn.ffn_sparse_forward_noalloc(dev.x, dev.w_gate, dev.w_up, dev.w_down_t, t, y)
    assert gu.rel_err(y.cpu().numpy(), gu.run_oracle(inp, t).y) <= 3e-5
    assert np.isfinite(y.cpu().numpy()).all()


@pytest.mark.parametrize("shape", [(256, 8, 8198, 4136), (100, 264, 300, 800)],
                         ids=["smaller pass, larger layout", "z in a region of its own"])
def test_wide_stays_in_the_workspace(gu, shape):
    """Ranks near and above d_ff / 2: z's partial copies do not fit where zval goes later.  Nothing
    behind the workspace is written, and the tokens of both ends of a pass are right."""
    import torch
    from paper_2609_31975_amd import ffn
    T, d, d_ff, r = shape
    t, n, guard = 1.6, ffn.workspace_bytes(*shape), 8 << 20
    inp = wl.make_inputs(606, T, d, d_ff, r=r, wdt=BF16)
    dev = gu.DevInputs(inp)
    buf = torch.full((n + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    buf[:n].zero_()
    y = torch.full((T, d), float("nan"), device="cuda")
    ffn.ffn_lopa_sparse_forward(dev.x, dev.lopa_a, dev.lopa_b, dev.w_up, dev.w_down_t, t, y, buf[:n])
    assert bool((buf[n:] == 0xA5).all())
    sel = [0, 15, T // 2 - 1, T // 2, T - 1]
    res = gu.run_oracle(inp, t, x=inp.x[sel])
    gu.check_parity(res, y.cpu().numpy()[sel], None, None, t, BF16, what=str(shape))


@pytest.mark.parametrize("wdt", [BF16, I8], ids=["bf16", "i8"])
def test_wide_full_form_with_partial_copies_of_z(gu, wdt):
    """Rows long enough that z comes in several partial copies, which the norm adds and clears."""
    T, d, d_ff, r, t = 150, 1552, 1500, 48, 2.0
    inp = wl.make_inputs(608, T, d, d_ff, r=r, wdt=wdt)
    form = gu.Form(act=1, silu_up=True, form=wl.make_form(608, d, d_ff, r), use_g=True, rms_norm=True, use_gain=True)
    dev = gu.DevInputs(inp)
    y = gu.run_gpu_q(dev, t, form=form)[0] if wdt == I8 else gu.run_gpu_ex(dev, t, form)[0]
    res = gu.run_oracle(inp, t, form=form)
    gu.check_parity(res, y, None, None, t, BF16, what=f"w{wdt}")
    assert gu.rel_err(y, res.y) <= 3e-5


# more than 64 tokens, and 33..64 of them; also fp32 weights on their matrix-core kernels
KINDS = [(100, 264, 1000, 40, BF16), (140, 264, 1000, 0, BF16), (40, 2304, 14300, 0, BF16), (16, 264, 1000, 0, wl.F32),
         (40, 264, 1000, 40, wl.F32)]


@pytest.mark.parametrize("shape", KINDS, ids=lambda s: "T%d_d%d_dff%d_r%d_w%d" % s)
def test_nothing_active(gu, shape):
    T, d, d_ff, r, wdt = shape
    y = gu.run_gpu(gu.DevInputs(wl.make_inputs(609, T, d, d_ff, r=r, wdt=wdt)), 1e30)[0]
    assert (y == 0).all()


@pytest.mark.parametrize("shape", KINDS, ids=lambda s: "T%d_d%d_dff%d_r%d_w%d" % s)
def test_nan_row_of_an_active_neuron(gu, shape):
    """NaN across the W_up row of a neuron that token 0 activates: NaN in the outputs of the tokens
    that activate it; the others' are right or NaN."""
    T, d, d_ff, r, wdt = shape
    t = 1.0
    inp = wl.make_inputs(610, T, d, d_ff, r=r, wdt=wdt)
    sel = sorted({0, 1, 7, T // 2, T - 1})
    res = gu.run_oracle(inp, t, x=inp.x[sel])
    clear = res.active[0] & ~(np.abs(res.h - t) < gu.BAND).any(0)
    i = int(np.flatnonzero(clear)[clear.sum() // 2])
    inp.w_up[i] = np.uint16(0x7FC0) if wdt == BF16 else np.float32(np.nan)
    y = gu.run_gpu(gu.DevInputs(inp), t)[0]
    for k, tau in enumerate(sel):
        row, ref = y[tau].astype(np.float64), np.asarray(res.y[k], np.float64)
        if res.active[k, i]:
            assert np.isnan(row).all(), tau
        else:
            assert np.isnan(row).all() or np.max(np.abs(row - ref)) <= gu.TOL[wdt] * np.max(np.abs(ref)), tau


@pytest.mark.parametrize("shape", KINDS, ids=lambda s: "T%d_d%d_dff%d_r%d_w%d" % s)
def test_graph_replay_and_two_streams(gu, shape):
    """Replays of a captured call, with other eager work between them, and calls on two streams at once
    with a workspace each, give the eager result."""
    import torch
    from paper_2609_31975_amd import ffn
    T, d, d_ff, r, wdt = shape
    t = 1.3
    dev = gu.DevInputs(wl.make_inputs(611, T, d, d_ff, r=r, wdt=wdt))
    wss = [ffn.alloc_workspace(T, d, d_ff, r) for _ in range(2)]
    ys = [torch.empty((T, d), device="cuda") for _ in range(2)]

    def call(k):
        if r:
            ffn.ffn_lopa_sparse_forward(dev.x, dev.lopa_a, dev.lopa_b, dev.w_up, dev.w_down_t, t, ys[k], wss[k])
        else:
            ffn.ffn_sparse_forward(dev.x, dev.w_gate, dev.w_up, dev.w_down_t, t, ys[k], wss[k])

    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    with torch.cuda.stream(streams[0]):
        call(0)
    torch.cuda.synchronize()
    eager = ys[0].cpu().numpy()
    assert np.isfinite(eager).all() and eager.any()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=streams[0]):
        call(0)
    other = torch.randn(1 << 20, device="cuda")
    for rep in range(3):
        ys[0].fill_(float("nan"))
        other.mul_(1.0001)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert gu.rel_err(ys[0].cpu().numpy(), eager) < 1e-6, f"replay {rep}"
    for rep in range(5):
        for y in ys:
            y.fill_(float("nan"))
        torch.cuda.synchronize()
        for k in range(2):
            with torch.cuda.stream(streams[k]):
                call(k)
        torch.cuda.synchronize()
        for k in range(2):
            assert gu.rel_err(ys[k].cpu().numpy(), eager) < 1e-6, f"rep {rep} stream {k}"
    del graph
