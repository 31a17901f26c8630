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


def test_a_smaller_workspace_still_serves():
    x = _gpu(_x(2, 900_001, (806,)))
    st = [("fir", _gpu(design.fir_lowpass(255, 9000.0, 48000.0).astype(np.float32))), ("sos", _gpu(_eq(6, 2)))]
    y, V = _prepared_run(x, st)
    assert V > 0
    y2, V2 = _prepared_run(x, st, ws_cut=256)
    assert V2 == 0 and _same(y2, _scan(x, st))
    assert_close(_cpu(y2), _cpu(y).astype(np.float64), TOL_IIR_F32, "scan against blocks")


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
    assert _same(tfx.chain(xb, st), want_b)
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
    for x, want in ((xc, got_c), (xb, want_b), (xb, want_b), (xc, got_c), (xb, want_b), (xc, got_c)):
        lib.call("tfx_chain_run", x.data_ptr(), y.data_ptr(), C, N, N, N, arr, len(desc), 0, None, ws.data_ptr(),
                 nb.value, sp)
        assert _same(y, want)


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
        assert _same(y, tfx.chain(x, st))
