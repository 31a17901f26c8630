"""Short-memory chains: an FFT FIR with a cascade whose response dies out
within 8192 samples runs as one FIR on 16384-point blocks.  Against the FP64
oracle over every cascade length and the edges of the tiles; and against the
scan (which a call that asks for checkpoints always takes), bit for bit, where
the chain must fall back to it: resonances that ring on, FP64-carry sections,
unstable ones, and samples that are not finite."""
import numpy as np
import pytest
import torch

import paper_2504_08624_amd as tfx
from paper_2504_08624_amd import design, lib, signals
from paper_2504_08624_amd.functional import _stages
from oracle import oracle as O
from tests.metrics import TOL_FIR_F32, TOL_IIR_F32, assert_close

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL_GRAD = 1e-4    # every gradient's bar, relative over each tensor
WORK = 10_000_000  # samples times sections from which the form is taken


def _x(C, N, key, sigma=0.1):
    return signals.to_f32(np.stack([signals.white(N, (*key, c), sigma) for c in range(C)]).reshape(C, N))


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _cpu(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def _eq(S, seed, lo=600.0):
    g = signals.rng(801, S, seed)
    return np.concatenate([design.peaking(f, q, d, 48000.0) for f, q, d in
                           zip(np.geomspace(lo, 15000.0, S), g.uniform(0.7, 2.0, S), g.uniform(-9.0, 9.0, S))]
                          ).astype(np.float32)


def _scan(x, stages):
    return tfx.chain(x, stages, return_ckpt=True)[0]


def _same(a, b):
    return torch.equal(torch.nan_to_num(a, nan=1e30), torch.nan_to_num(b, nan=1e30))


@pytest.mark.parametrize("S", [1, 2, 5, 6, 7, 8])
@pytest.mark.parametrize("M", [49, 255, 1025, 2049])
def test_against_oracle(S, M):
    C = 3
    N = WORK // (S * C) + 17
    print("short chain S=%d M=%d N=%d" % (S, M, N), flush=True)
    x = _x(C, N, (802, S, M))
    h = design.fir_lowpass(M, 9000.0, 48000.0).astype(np.float32)
    sec = _eq(S, M)
    stages = [("fir", _gpu(h)), ("sos", _gpu(sec))]
    xg = _gpu(x)
    y = tfx.chain(xg, stages)
    ref = O.chain(x, [("fir", h), ("sos", sec)])
    # one filter on one transform: its own error is the FIR's, not the recursion's
    assert_close(_cpu(y), ref, TOL_FIR_F32, "S=%d M=%d" % (S, M))
    assert not torch.equal(y, _scan(xg, stages))           # the form under test did run


@pytest.mark.parametrize("extra", [-1, 0, 1, 63, 64])
def test_tile_edges(extra):
    """Signals that end within a sample of a tile or of a pair of tiles: with
    V the chain's memory from the workspace header, tiles of 16384 - V."""
    h = design.fir_lowpass(200, 9000.0, 48000.0).astype(np.float32)
    sec = _eq(8, 1)
    C = 5
    st = [("fir", _gpu(h)), ("sos", _gpu(sec))]
    _, V = _prepared_run(_gpu(_x(C, 300_000, (803,))), st)
    T = 16384 - V
    for k in (17, 18):
        N = k * T + extra
        x = _x(C, N, (804, k, extra + 1))
        assert C * N * 8 >= WORK
        assert_close(_cpu(tfx.chain(_gpu(x), st)), O.chain(x, [("fir", h), ("sos", sec)]), TOL_FIR_F32,
                     "%d tiles %+d" % (k, extra))


def _prepared_run(x, stages, ws_cut=0):
    """chain_prepare + chain_run; returns y and the memory V (0: not short)."""
    C, N = x.shape
    kept, desc = _stages(stages, torch.device(DEV))
    arr = lib.stage_array(desc)
    nb = lib.size_out()
    lib.call("tfx_chain_workspace_size", C, N, arr, len(desc), 0, nb)
    ws = torch.zeros(nb.value, dtype=torch.uint8, device=DEV)
    y = torch.empty_like(x)
    sp = torch.cuda.current_stream().cuda_stream
    lib.call("tfx_chain_prepare", C, N, arr, len(desc), 0, ws.data_ptr(), nb.value - ws_cut, sp)
    lib.call("tfx_chain_run", x.data_ptr(), y.data_ptr(), C, N, N, N, arr, len(desc), 0, None, ws.data_ptr(),
             nb.value - ws_cut, sp)
    torch.cuda.synchronize()
    v = int(ws[:64].view(torch.int32)[4])
    assert v == 0 or v % 64 == 1
    return y, max(v - 1, 0)


@pytest.mark.parametrize("sec", [
    pytest.param(np.array([[1, -1.99, 1, -1.995, 0.9956]] * 2, np.float32), id="rings on"),
    pytest.param(np.array([[0.1, 0.2, 0.1, -1.2, 0.9999]] * 2, np.float32), id="fp64 carry"),
    pytest.param(np.array([[1, 0, 0, -2.0, 1.0001]] * 2, np.float32), id="unstable"),
    pytest.param(np.array([[1, 0, 0, float("nan"), 0.5]] * 2, np.float32), id="nan"),
])
def test_other_chains_run_as_before(sec):
    x = _gpu(_x(2, 2_600_000, (805,)))
    st = [("fir", _gpu(design.fir_lowpass(255, 9000.0, 48000.0).astype(np.float32))), ("sos", _gpu(sec))]
    y, V = _prepared_run(x, st)
    assert V == 0
    want = _scan(x, st)
    if sec[0, 4] < 0.999:
        assert _same(y, want) and _same(tfx.chain(x, st), y)
    else:
        # poles this close to the circle (or beyond it) have no finite look-back
        # depth: the nearest finished tile ends a look-back, and two runs of the
        # scan itself differ in their last bits
        k = 30_000                                             # before the unstable chain overflows
        assert_close(_cpu(y[:, :k]), _cpu(want[:, :k]).astype(np.float64), TOL_IIR_F32, "two runs of the scan")
        assert bool(torch.isfinite(y[:, -1]).all()) == bool(torch.isfinite(want[:, -1]).all())


@pytest.mark.parametrize("cmp,dt", [("bf16", torch.bfloat16), ("f16", torch.float16)])
@pytest.mark.parametrize("S,M", [(1, 5), (2, 255), (6, 1023), (8, 2049)])
def test_rounded_operands(cmp, dt, S, M):
    """bf16 and fp16 operands: the oracle on the rounded signal and taps, and the
    scan behind the matrix-core FIR."""
    C = 3
    N = WORK // (S * C) + 17
    x = _x(C, N, (820, S, M))
    h = design.fir_lowpass(M, 9000.0, 48000.0).astype(np.float32)
    sec = _eq(S, M)
    st = [("fir", _gpu(h)), ("sos", _gpu(sec))]
    xg = _gpu(x)
    y = tfx.chain(xg, st, compute=cmp)
    xr, hr = _cpu(xg.to(dt).float()), _cpu(st[0][1].to(dt).float())
    assert_close(_cpu(y), O.chain(xr, [("fir", hr), ("sos", sec)]), TOL_FIR_F32, "%s S=%d M=%d" % (cmp, S, M))
    scan = tfx.chain(xg, st, compute=cmp, return_ckpt=True)[0]
    assert not torch.equal(y, scan)
    assert_close(_cpu(y), _cpu(scan).astype(np.float64), TOL_IIR_F32, "against the scan")
    if cmp == "f16":                                       # over fp16's range: infinite there, and done again
        xg[1, 200_000] = 7e4
        want = tfx.chain(xg, st, compute=cmp, return_ckpt=True)[0]
        got = tfx.chain(xg, st, compute=cmp)
        lo, hi = 200_000 - 9000, 200_000 + 9000 + 30 * 3072
        assert _same(got[:, :lo], want[:, :lo]) and _same(got[:, hi:], want[:, hi:])
        assert not bool(torch.isfinite(got[1, 200_000])) and not bool(torch.isfinite(want[1, 200_000]))


def test_a_smaller_workspace_still_serves():
    x = _gpu(_x(2, 900_001, (806,)))
    st = [("fir", _gpu(design.fir_lowpass(255, 9000.0, 48000.0).astype(np.float32))), ("sos", _gpu(_eq(6, 2)))]
    y, V = _prepared_run(x, st)
    assert V > 0
    y2, V2 = _prepared_run(x, st, ws_cut=256)
    assert V2 == 0 and _same(y2, _scan(x, st))
    assert_close(_cpu(y2), _cpu(y).astype(np.float64), TOL_IIR_F32, "scan against blocks")


def test_prepare_and_run_with_workspaces_of_two_sizes():
    """A prepare without the room for the short-memory tables, on a buffer in which
    another filter's lie, and a run that has the room (and the other way round):
    the scan, of the filter that was prepared last."""
    C, N = 2, 900_001
    x = _gpu(_x(C, N, (830,)))
    filters = []
    for k in (0, 1):
        st = [("fir", _gpu(design.fir_lowpass(255 - 40 * k, 9000.0 - 3000.0 * k, 48000.0).astype(np.float32))),
              ("sos", _gpu(_eq(6, 10 + k)))]
        kept, desc = _stages(st, torch.device(DEV))
        filters.append((st, kept, lib.stage_array(desc), len(desc)))
    nb = lib.size_out()
    lib.call("tfx_chain_workspace_size", C, N, filters[0][2], filters[0][3], 0, nb)
    ws = torch.zeros(nb.value, dtype=torch.uint8, device=DEV)
    y = torch.empty_like(x)
    sp = torch.cuda.current_stream().cuda_stream

    def call(k, cut_prepare, cut_run):
        _, _, arr, n = filters[k]
        lib.call("tfx_chain_prepare", C, N, arr, n, 0, ws.data_ptr(), nb.value - cut_prepare, sp)
        for _ in range(2):
            lib.call("tfx_chain_run", x.data_ptr(), y.data_ptr(), C, N, N, N, arr, n, 0, None, ws.data_ptr(),
                     nb.value - cut_run, sp)
        return y

    blocks = call(0, 0, 0).clone()
    assert not _same(blocks, _scan(x, filters[0][0]))
    assert _same(call(1, 256, 0), _scan(x, filters[1][0]))     # filter 0's tables still lie there
    assert _same(call(0, 0, 256), _scan(x, filters[0][0]))
    assert _same(call(0, 0, 0), blocks)


@pytest.mark.parametrize("M", [255, 1500])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf"), 3e38])
def test_values_that_are_not_finite(bad, M):
    """The run that meets one is done again by the scan, and the next run on
    the same workspace is a block run again."""
    C, N = 3, 1_700_011
    xb = _gpu(_x(C, N, (807,)))
    xc = xb.clone()
    if abs(bad) < 4e38 and np.isfinite(bad):
        xb[1, 800_000:800_400] = bad                        # finite, but its sums overflow
    else:
        xb[1, 800_000] = bad
    h = np.ones(M, np.float32) if np.isfinite(bad) else design.fir_lowpass(M, 9000.0, 48000.0).astype(np.float32)
    st = [("fir", _gpu(h)), ("sos", _gpu(_eq(2, 3)))]
    want_b, want_c = _scan(xb, st), _scan(xc, st)
    assert not bool(torch.isfinite(want_b).all())
    got_c = tfx.chain(xc, st)

    # how many tiles behind it a bad sample reaches is up to which of the scan's
    # records are out when a tile looks: two runs of the scan may differ there
    def same_b(y):
        lo, hi = 800_000 - 40_000, 800_000 + 40_000 + 30 * 3072
        return _same(y[:, :lo], want_b[:, :lo]) and _same(y[:, hi:], want_b[:, hi:]) and \
            _same(torch.isfinite(y[:, 800_000:802_000]).float(), torch.isfinite(want_b[:, 800_000:802_000]).float())

    assert same_b(tfx.chain(xb, st))
    assert_close(_cpu(got_c), _cpu(want_c).astype(np.float64), TOL_IIR_F32, "clean")
    # several runs on one prepared workspace
    kept, desc = _stages(st, torch.device(DEV))
    arr = lib.stage_array(desc)
    nb = lib.size_out()
    lib.call("tfx_chain_workspace_size", C, N, arr, len(desc), 0, nb)
    ws = torch.zeros(nb.value, dtype=torch.uint8, device=DEV)
    y = torch.empty_like(xb)
    sp = torch.cuda.current_stream().cuda_stream
    lib.call("tfx_chain_prepare", C, N, arr, len(desc), 0, ws.data_ptr(), nb.value, sp)
    for x, bad_run in ((xc, 0), (xb, 1), (xb, 1), (xc, 0), (xb, 1), (xc, 0)):
        lib.call("tfx_chain_run", x.data_ptr(), y.data_ptr(), C, N, N, N, arr, len(desc), 0, None, ws.data_ptr(),
                 nb.value, sp)
        assert same_b(y) if bad_run else _same(y, got_c)


def test_graph_replays():
    C, N = 2, 1_300_003
    st = [("fir", _gpu(design.fir_lowpass(300, 9000.0, 48000.0).astype(np.float32))), ("sos", _gpu(_eq(4, 4)))]
    x = _gpu(_x(C, N, (808,)))
    kept, desc = _stages(st, torch.device(DEV))
    arr = lib.stage_array(desc)
    nb = lib.size_out()
    lib.call("tfx_chain_workspace_size", C, N, arr, len(desc), 0, nb)
    ws = torch.zeros(nb.value, dtype=torch.uint8, device=DEV)
    y = torch.empty_like(x)
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        lib.call("tfx_chain_prepare", C, N, arr, len(desc), 0, ws.data_ptr(), nb.value, s.cuda_stream)
        lib.call("tfx_chain_run", x.data_ptr(), y.data_ptr(), C, N, N, N, arr, len(desc), 0, None, ws.data_ptr(),
                 nb.value, s.cuda_stream)
    for k in range(4):
        x.copy_(_gpu(_x(C, N, (809, k))))
        if k == 2:
            x[0, 5] = float("nan")
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        w = tfx.chain(x, st)
        assert _same(y, w) if k != 2 else _same(y[:, 200_000:], w[:, 200_000:]) and bool(torch.isnan(y[0, 5]))


# ------------------------------------------------------------------ the adjoint

def _grads(x, g, coefs, kinds, need=None):
    """Autograd's gradients of the chain (None where not needed)."""
    need = need or [True] * (1 + len(coefs))
    ts = [t.clone().requires_grad_(n) for t, n in zip([x] + coefs, need)]
    tfx.chain(ts[0], list(zip(kinds, ts[1:]))).backward(g)
    return [t.grad for t in ts]


def _scan_backward(x, g, stages):
    """The adjoint by the scan: checkpoints, and a workspace without the room the
    other form wants."""
    _, ck = tfx.chain(x, stages, return_ckpt=True)
    C, N = x.shape
    kept, desc = _stages(stages, torch.device(DEV))
    arr = lib.stage_array(desc)
    nb = lib.size_out()
    lib.call("tfx_chain_backward_workspace_size", C, N, arr, len(desc), 0, nb)
    ws = torch.zeros(nb.value, dtype=torch.uint8, device=DEV)
    gx = torch.empty_like(x)
    gs = [torch.empty_like(t) for t in kept]
    lib.call("tfx_chain_backward", x.data_ptr(), g.data_ptr(), gx.data_ptr(), C, N, N, N, N, arr, len(desc), 0,
             ck.data_ptr(), lib.pointer_array([t.data_ptr() for t in gs]), ws.data_ptr(), nb.value - 256,
             torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return [gx] + gs


def _rel(a, b):
    return np.linalg.norm(_cpu(a).astype(np.float64).ravel() - np.ravel(b)) / np.linalg.norm(b)


@pytest.mark.parametrize("S", [1, 2, 7, 8])
@pytest.mark.parametrize("M", [49, 1025, 2049])
def test_gradients_against_oracle(S, M):
    C = 3
    N = WORK // (S * C) + 33
    print("short adjoint S=%d M=%d N=%d" % (S, M, N), flush=True)
    x = _x(C, N, (811, S, M))
    h = design.fir_lowpass(M, 9000.0, 48000.0).astype(np.float32)
    sec = _eq(S, M)
    # a residual correlated with the output, as a loss gives
    g = (np.roll(x, 3, axis=1) + 0.1 * _x(C, N, (812, S, M), 1.0)).astype(np.float32)
    got = _grads(_gpu(x), _gpu(g), [_gpu(h), _gpu(sec)], ["fir", "sos"])
    rgx, (rgh, rgs) = O.chain_backward(g, x, [("fir", h), ("sos", sec)])
    assert_close(_cpu(got[0]), rgx, TOL_FIR_F32, "dL/dx")
    for a, b, what in ((got[1], rgh, "dL/dh"), (got[2], rgs, "dL/dsos")):
        e = _rel(a, b)
        print("%s rel err %.2e" % (what, e), flush=True)
        assert e <= TOL_GRAD, "%s rel err %.3e" % (what, e)


def test_gradients_of_several_stages():
    """Two FIR and two section stages in mixed order, all gradients and some."""
    C, N = 2, 1_300_001
    x, g = _x(C, N, (813,)), _x(C, N, (814,))
    g = (g + np.roll(x, 1, axis=1)).astype(np.float32)
    coefs = [_eq(2, 1), design.fir_lowpass(100, 9000.0, 48000.0).astype(np.float32), _eq(3, 2),
             design.fir_lowpass(33, 12000.0, 48000.0).astype(np.float32)]
    kinds = ["sos", "fir", "sos", "fir"]
    xg, gg, cg = _gpu(x), _gpu(g), [_gpu(c) for c in coefs]
    got = _grads(xg, gg, cg, kinds)
    rgx, refs = O.chain_backward(g, x, list(zip(kinds, coefs)))
    assert_close(_cpu(got[0]), rgx, TOL_FIR_F32, "dL/dx")
    for i, (a, b) in enumerate(zip(got[1:], refs)):
        assert _rel(a, b) <= TOL_GRAD, "stage %d" % i
    some = _grads(xg, gg, cg, kinds, [True, False, True, False, False])
    assert torch.equal(some[0], got[0]) and torch.equal(some[2], got[2]) and some[1] is None
    only = _grads(xg, gg, cg, kinds, [True, False, False, False, False])
    assert torch.equal(only[0], got[0])
    coef = _grads(xg, gg, cg, kinds, [False, True, True, True, True])
    assert all(torch.equal(a, b) for a, b in zip(coef[1:], got[1:]))


@pytest.mark.parametrize("M", [255, 1500])
@pytest.mark.parametrize("where", ["x", "g"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_gradients_of_values_that_are_not_finite(bad, where, M):
    C, N = 3, 1_700_011
    x, g = _gpu(_x(C, N, (815,))), _gpu(_x(C, N, (816,)))
    h, sec = _gpu(design.fir_lowpass(M, 9000.0, 48000.0).astype(np.float32)), _gpu(_eq(2, 3))
    clean = _grads(x, g, [h, sec], ["fir", "sos"])
    (x if where == "x" else g)[1, 900_000] = bad
    got = _grads(x, g, [h, sec], ["fir", "sos"])
    want = _scan_backward(x, g, [("fir", h), ("sos", sec)])
    for a, b, c in zip(got[1:], want[1:], clean[1:]):
        assert _same(torch.isfinite(a).float(), torch.isfinite(b).float()) and bool(torch.isfinite(c).all())
    assert not bool(torch.isfinite(got[1]).all())
    # how many tiles before it a bad sample of g reaches is up to which of the
    # scan's records are out when a tile looks: between 30 tiles before and the
    # next block after it two runs of the scan may differ
    a, b = got[0], want[0]
    lo, hi = 900_000 - 30 * 3072, 900_000 + 3 * 8192
    assert _same(a[2], b[2]) and _same(a[:, :lo], b[:, :lo]) and _same(a[:, hi:], b[:, hi:])
    assert bool(torch.isfinite(a[1, 900_000])) == bool(torch.isfinite(b[1, 900_000])) == (where == "x")


def test_gradients_of_other_chains_and_explicit_checkpoints():
    x, g = _gpu(_x(2, 2_600_000, (817,))), _gpu(_x(2, 2_600_000, (818,)))
    h = _gpu(design.fir_lowpass(255, 9000.0, 48000.0).astype(np.float32))
    rings = _gpu(np.array([[1, -1.99, 1, -1.995, 0.9956]] * 2, np.float32))
    for sec, short in ((rings, False), (_gpu(_eq(2, 5)), True)):
        st = [("fir", h), ("sos", sec)]
        want = _scan_backward(x, g, st)
        got = _grads(x, g, [h, sec], ["fir", "sos"])
        gx, gs = tfx.chain_backward(x, g, st, _scan_ckpt(x, st))
        for a, b, c in zip(got, want, [gx] + gs):
            if short:                          # (two runs of the scan differ in their last bits for the other)
                assert torch.equal(a, c) and not torch.equal(a, b)
            for v in (a, c):
                assert _rel(v, _cpu(b).astype(np.float64)) <= 2 * TOL_GRAD


def _scan_ckpt(x, stages):
    return tfx.chain(x, stages, return_ckpt=True)[1]


def test_gradient_sums_over_many_tiles():
    """Many equal rows, a sine that a few bins of the transform hold: the sums over
    tiles round alike, and their error is that of a short fp32 sum however many
    tiles there are (256 a workgroup here; fp32 alone would be off by 1e-6 and more)."""
    rows, N = 131_072, 9_600
    h = design.fir_lowpass(101, 9000.0, 48000.0).astype(np.float32)
    sec = _eq(2, 7)
    n = np.arange(N)
    worst = 0.0
    for amp in (0.1, 0.125, 0.16, 0.19):
        x1 = (amp * np.sin(2 * np.pi * 700 * n / 16384 + 0.3)).astype(np.float32)[None]
        g1 = (0.7 * amp * np.sin(2 * np.pi * 700 * n / 16384 + 1.1)).astype(np.float32)[None]
        _, (rgh, rgs) = O.chain_backward(g1, x1, [("fir", h), ("sos", sec)])
        x, g = _gpu(x1).expand(rows, N).contiguous(), _gpu(g1).expand(rows, N).contiguous()
        got = _grads(x, g, [_gpu(h), _gpu(sec)], ["fir", "sos"], [False, True, True])
        del x, g
        eh, es = _rel(got[1], rows * rgh), _rel(got[2], rows * rgs)
        print("sums over %d rows: dL/dh %.2e dL/dsos %.2e" % (rows, eh, es), flush=True)
        worst = max(worst, eh, es)
    # 8 roundings of 2^-24 in a row (4.8e-7), and the transforms' own
    assert worst <= 1e-6


@pytest.mark.parametrize("C,N,S,lo,blocks", [
    pytest.param(4096, 1024, 4, 600.0, False, id="rows far shorter than a block"),
    pytest.param(1000, 15_000, 2, 6000.0, True, id="rows of one tile"),
    pytest.param(1000, 15_000, 2, 200.0, False, id="rows of just over one tile, known on the device"),
    pytest.param(1001, 15_000, 6, 200.0, True, id="rows of just over one tile, a longer cascade"),
])
def test_rows_that_are_worth_blocks(C, N, S, lo, blocks):
    """The form by the row's length, the cascade's and the chain's memory."""
    x = _gpu(_x(8, N, (831, N, S))).repeat((C + 7) // 8, 1)[:C].contiguous()
    h, sec = design.fir_lowpass(101, 9000.0, 48000.0).astype(np.float32), _eq(S, 3, lo)
    st = [("fir", _gpu(h)), ("sos", _gpu(sec))]
    assert C * N * S >= WORK
    y, V = _prepared_run(x, st)
    assert (V > 0) == blocks
    ref = O.chain(_cpu(x[:8]), [("fir", h), ("sos", sec)])
    assert_close(_cpu(y[:8]), ref, TOL_FIR_F32 if blocks else TOL_IIR_F32, "first rows")
    assert_close(_cpu(y[C - C % 8 - 8:C - C % 8]), ref, TOL_FIR_F32 if blocks else TOL_IIR_F32, "last rows")
    if blocks:
        assert not torch.equal(y, _scan(x, st))
    else:
        assert torch.equal(y, _scan(x, st))
    # the adjoint follows whichever form the forward took
    g = torch.roll(x, 3, 1)
    got = _grads(x[:C - C % 8], g[:C - C % 8], [_gpu(h), _gpu(sec)], ["fir", "sos"])
    rgx, (rgh, rgs) = O.chain_backward(_cpu(g[:8]), _cpu(x[:8]), [("fir", h), ("sos", sec)])
    assert_close(_cpu(got[0][-8:]), rgx, TOL_IIR_F32, "dL/dx")
    assert _rel(got[1], C // 8 * rgh) <= TOL_GRAD and _rel(got[2], C // 8 * rgs) <= TOL_GRAD


def _train_calls(x, g, stages, cmp=0, cut=0):
    """tfx_chain_train and tfx_chain_train_backward (fp32, its workspace cut bytes
    short of the query), checkpoints from a buffer of NaN: y, the gradients and
    the checkpoints as the forward left them."""
    C, N = x.shape
    kept, desc = _stages(stages, torch.device(DEV))
    arr, n = lib.stage_array(desc), len(desc)
    S = sum(k for kind, k, _ in desc if kind == lib.STAGE_SOS)
    nb, nbb = lib.size_out(), lib.size_out()
    lib.call("tfx_chain_workspace_size", C, N, arr, n, cmp, nb)
    lib.call("tfx_chain_backward_workspace_size", C, N, arr, n, 0, nbb)
    ws = torch.empty(nb.value, dtype=torch.uint8, device=DEV)
    wsb = torch.empty(nbb.value, dtype=torch.uint8, device=DEV)
    y, gx, gs = torch.empty_like(x), torch.empty_like(x), [torch.empty_like(t) for t in kept]
    ck = torch.full((C, (N + 3071) // 3072, S, 2), float("nan"), device=DEV)
    sp = torch.cuda.current_stream().cuda_stream
    lib.call("tfx_chain_train", x.data_ptr(), y.data_ptr(), C, N, N, N, arr, n, cmp, ck.data_ptr(), ws.data_ptr(),
             nb.value, sp)
    left = ck.clone()
    lib.call("tfx_chain_train_backward", x.data_ptr(), g.data_ptr(), gx.data_ptr(), C, N, N, N, N, arr, n, 0,
             ck.data_ptr(), lib.pointer_array([t.data_ptr() for t in gs]), wsb.data_ptr(), nbb.value - cut, sp)
    torch.cuda.synchronize()
    return y, [gx] + gs, left


@pytest.mark.parametrize("M", [5, 255])
def test_checkpoints_of_rounded_operands(M):
    """A training forward with bf16 operands writes its checkpoints: the adjoint, in
    fp32, may take a form that cannot do without them (5 taps: a direct FIR)."""
    C, N = 3, 1_700_011
    x, g = _gpu(_x(C, N, (832, M))), _gpu(_x(C, N, (833, M)))
    st = [("fir", _gpu(design.fir_lowpass(M, 9000.0, 48000.0).astype(np.float32))), ("sos", _gpu(_eq(3, 4)))]
    y, ck = tfx.chain(x, st, compute="bf16", return_ckpt=True)
    want = tfx.chain_backward(x, g, st, ck)
    got_y, got, left = _train_calls(x, g, st, cmp=lib.COMPUTE["bf16"])
    assert torch.equal(got_y, y) and torch.equal(left, ck)
    for a, b in zip(got, [want[0]] + want[1]):
        assert _rel(a, _cpu(b).astype(np.float64)) <= TOL_GRAD


@pytest.mark.parametrize("k", [0, 1, 2])
@pytest.mark.parametrize("col", [0, 3, 4])
def test_a_nan_in_one_section(k, col):
    """Whichever section holds it, such a chain is none of short memory."""
    sec = _eq(3, 6)
    sec[k, col] = np.nan
    x = _gpu(_x(2, 2_600_000, (834,)))
    st = [("fir", _gpu(design.fir_lowpass(255, 9000.0, 48000.0).astype(np.float32))), ("sos", _gpu(sec))]
    y, V = _prepared_run(x, st)
    assert V == 0 and bool(torch.isnan(y[:, 2:]).all())     # (a2 first counts two samples on)


def _resonance(theta, r, n):
    """n equal sections with poles r e^(+-i theta), about unit gain there."""
    return np.array([[2 * (1 - r) * np.sin(theta), 0.0, 0.0, -2 * r * np.cos(theta), r * r]] * n, np.float32)


@pytest.mark.parametrize("theta,r,n,blocks", [
    (0.3, 0.9965, 2, True), (1.5, 0.9962, 3, True), (0.3, 0.996, 4, True), (1.5, 0.9968, 2, False),
    (0.3, 0.9965, 4, False)])
def test_memory_at_its_limit(theta, r, n, blocks):
    """Narrow resonances and repeated poles whose memory is all but 8192 samples, and
    just over: output and every gradient.  (The gradient's responses, sums of
    h delayed, die out more slowly than h itself.)"""
    C = 2
    N = WORK // (n * C) + 501
    x = _x(C, N, (835, n))
    h, sec = design.fir_lowpass(49, 9000.0, 48000.0).astype(np.float32), _resonance(theta, r, n)
    st = [("fir", _gpu(h)), ("sos", _gpu(sec))]
    y, V = _prepared_run(_gpu(x), st)
    print("memory %d of theta %g r %g, %d sections" % (V, theta, r, n), flush=True)
    assert 7500 <= V <= 8192 if blocks else V == 0
    assert_close(_cpu(y), O.chain(x, [("fir", h), ("sos", sec)]), TOL_FIR_F32 if blocks else TOL_IIR_F32, "output")
    g = (np.roll(x, 3, axis=1) + 0.1 * _x(C, N, (836, n), 1.0)).astype(np.float32)
    got = _grads(_gpu(x), _gpu(g), [_gpu(h), _gpu(sec)], ["fir", "sos"])
    rgx, (rgh, rgs) = O.chain_backward(g, x, [("fir", h), ("sos", sec)])
    eh, es = _rel(got[1], rgh), _rel(got[2], rgs)
    print("gradients: dL/dh %.2e dL/dsos %.2e" % (eh, es), flush=True)
    assert_close(_cpu(got[0]), rgx, TOL_FIR_F32 if blocks else TOL_IIR_F32, "dL/dx")
    assert eh <= TOL_GRAD and es <= TOL_GRAD


@pytest.mark.parametrize("kind", ["short", "fp64 carry", "rings on"])
@pytest.mark.parametrize("M", [255, 1500])
def test_lazy_checkpoints_and_a_backward_without_the_room(kind, M):
    """tfx_chain_train, whose short-memory form leaves the checkpoints out, and a
    backward call whose workspace has no room for that form's adjoint."""
    C, N = 2, 1_300_003
    x, g = _gpu(_x(C, N, (837, M))), _gpu(_x(C, N, (838, M)))
    sec = {"short": _eq(4, 8), "rings on": np.array([[1, -1.99, 1, -1.995, 0.9956]] * 4, np.float32),
           "fp64 carry": _resonance(1.0, 0.9995, 4)}[kind]
    st = [("fir", _gpu(design.fir_lowpass(M, 9000.0, 48000.0).astype(np.float32))), ("sos", _gpu(sec))]
    want = _scan_backward(x, g, st)
    for cut in (256, 0):
        _, got, left = _train_calls(x, g, st, cut=cut)
        assert bool(torch.isnan(left).any()) == (kind == "short")
        for a, b in zip(got, want):
            assert _rel(a, _cpu(b).astype(np.float64)) <= 2 * TOL_GRAD
