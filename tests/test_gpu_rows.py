"""Rows that start at any 4-byte boundary (16-byte tile accesses at each of the
four offsets, in and out), and cascades that return their final registers over
signals of one to many tiles, for every cascade length that has a form of its
own, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import paper_2504_08624_amd as tfx
from paper_2504_08624_amd import design, signals
from oracle import oracle as O
from tests.metrics import TOL_FIR_LOWP, TOL_IIR_F32, assert_close

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
T = 3072


def _x(C, N, key, sigma=0.1):
    return signals.to_f32(np.stack([signals.white(N, (*key, c), sigma) for c in range(C)]).reshape(C, N))


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _cpu(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def _eq(S, key):
    g = signals.rng(900, S, key)
    return np.concatenate([design.peaking(f, q, d, 48000.0) for f, q, d in
                           zip(np.geomspace(500.0, 15000.0, S), g.uniform(0.7, 2.0, S), g.uniform(-9.0, 9.0, S))]
                          ).astype(np.float32)


def _at(x, off):
    """x on the device with row 0 starting off floats behind a 16-byte boundary."""
    buf = torch.zeros(x.size + 8 + x.shape[0], dtype=torch.float32, device=DEV)
    v = buf[off:off + x.size].view(x.shape)
    v.copy_(_gpu(x))
    return v


@pytest.mark.parametrize("off", [0, 1, 2, 3])
@pytest.mark.parametrize("N", [T, 2 * T + 1, 3 * T - 1])
@pytest.mark.parametrize("form", ["sos4", "sos8", "sos12", "direct", "fft", "bf16"])
def test_row_offsets(off, N, form):
    x = _x(3, N, (901, N))
    S = {"sos4": 4, "sos8": 8, "sos12": 12}.get(form, 3)
    sec = _eq(S, 1)
    stages, tol, kw = [("sos", sec)], TOL_IIR_F32, {}
    if form in ("direct", "fft", "bf16"):
        stages.insert(0, ("fir", design.fir_lowpass(17 if form == "direct" else 201, 9000.0, 48000.0).astype(np.float32)))
    if form == "bf16":
        tol, kw = TOL_FIR_LOWP, {"compute": "bf16"}
    y = tfx.chain(_at(x, off), [(k, _gpu(c)) for k, c in stages], **kw)
    assert_close(_cpu(y), O.chain(x, stages), tol, "%s N=%d offset %d" % (form, N, off))
    if form != "bf16":
        xg, gg = _at(x, off), _at(x[::-1].copy(), (off + 1) % 4)
        st = [(k, _gpu(c)) for k, c in stages]
        _, ck = tfx.chain(xg, st, return_ckpt=True)
        gx, _ = tfx.chain_backward(xg, gg, st, ck)
        rgx, _ = O.chain_backward(x[::-1].copy(), x, stages)
        assert_close(_cpu(gx), rgx, TOL_IIR_F32, "adjoint %s N=%d offset %d" % (form, N, off))


@pytest.mark.parametrize("S", [1, 3, 6, 7, 8, 9])
@pytest.mark.parametrize("N", [1, T - 1, T, T + 1, 2 * T, 70 * T + 5])
def test_final_registers(S, N):
    C = 3
    x = _x(C, N, (902, S, N))
    sec = _eq(S, 2)
    s0 = (0.05 * signals.rng(903, S, N).standard_normal((C, S, 2))).astype(np.float32)
    y, so, ck = tfx.sos(_gpu(x), _gpu(sec), state_in=_gpu(s0), return_state=True, return_ckpt=True)
    ref, rs = O.sos(x, sec, state_in=s0, return_state=True)
    assert_close(_cpu(y), ref, TOL_IIR_F32, "S=%d N=%d" % (S, N))
    # a register is a difference of products of samples: its rounding goes by the
    # samples' size (0.1), not by its own
    assert np.max(np.abs(_cpu(so) - rs)) <= TOL_IIR_F32 * 0.1, "registers S=%d N=%d" % (S, N)
    # the registers carry on: the rest of a longer signal from them
    z = _x(C, 2 * T + 9, (904, S, N))
    y2 = tfx.sos(_gpu(z), _gpu(sec), state_in=so)
    ref2 = O.sos(np.concatenate([x, z], axis=1), sec, state_in=s0)[:, N:]
    assert_close(_cpu(y2), ref2, TOL_IIR_F32, "continued S=%d N=%d" % (S, N))


@pytest.mark.parametrize("S,tiles", [(8, 700), (6, 2400), (4, 31), (4, 33)])  # split, split, one launch, two
def test_final_registers_by_size(S, tiles):
    """Each side of the rules by which a call's tiles share a launch (6 channels:
    3 workgroups a tile); the last channel's last tile and its registers against
    the oracle on the signal's tail from the registers in front of it."""
    C, N = (6 if S > 4 else 4), tiles * T - 9
    tail = 5 * T + 11
    x = _x(C, N, (906, S, tiles))
    sec = _eq(S, 3)
    y, so = tfx.sos(_gpu(x), _gpu(sec), return_state=True)
    head = N - tail
    _, s0 = O.sos(x[-1:, max(0, head - 20 * T):head], sec, return_state=True)  # decays within a tile
    ref, rs = O.sos(x[-1:, head:], sec, state_in=s0, return_state=True)
    assert_close(_cpu(y)[-1:, head:], ref, TOL_IIR_F32, "tail S=%d tiles=%d" % (S, tiles))
    assert np.max(np.abs(_cpu(so)[-1:] - rs)) <= TOL_IIR_F32 * 0.1, "registers S=%d tiles=%d" % (S, tiles)


@pytest.mark.parametrize("taps", [0, 17, 201])
@pytest.mark.parametrize("q", [1.0, 400.0])  # 400: poles that the FP64-carry form takes
def test_stream_of_mixed_blocks(taps, q):
    """Blocks of one and of several tiles in turn on one workspace: the one-tile
    form, the split one, and the look-back's records from run to run."""
    C, sizes = 3, (1, 512, T, T + 1, 3 * T + 7, 5, 2 * T, 512)
    N = sum(sizes)
    x = _x(C, N, (905, taps))
    sec = np.concatenate([design.peaking(f, q, 6.0, 48000.0) for f in (4000.0, 8000.0, 15000.0)]).astype(np.float32)
    stages = [("sos", sec)]
    if taps:
        stages.insert(0, ("fir", design.fir_lowpass(taps, 9000.0, 48000.0).astype(np.float32)))
    stream = tfx.ChainStream([(k, _gpu(c)) for k, c in stages], C, max(sizes))
    for again in range(2):  # the second time from reset(), on records of the first
        n0, out = 0, []
        for b in sizes:
            out.append(_cpu(stream.process(_gpu(x[:, n0:n0 + b]))))
            n0 += b
        assert_close(np.concatenate(out, axis=1), O.chain(x, stages), TOL_IIR_F32, "taps %d q %g" % (taps, q))
        stream.reset()


@pytest.mark.parametrize("S,tiles", [(7, 933), (7, 934), (3, 9340)])
def test_final_registers_by_size_of_seven_and_three(S, tiles):
    """Either side of the rule at 7 sections (2800 workgroups), and 3, which keep to
    one launch, with registers coming in."""
    C, N = 6, tiles * T - 9
    x = _gpu(_x(C, 6 * T + 1, (907, S))).repeat(1, tiles // 6 + 1)[:, :N].contiguous()
    sec = _eq(S, 4)
    s0 = (0.05 * signals.rng(908, S).standard_normal((C, S, 2))).astype(np.float32)
    y, so = tfx.sos(x, _gpu(sec), state_in=_gpu(s0), return_state=True)
    tail = 25 * T + 11
    ref, rs = O.sos(_cpu(x[:, -tail:]), sec, return_state=True)      # the registers decay within a tile
    assert_close(_cpu(y[:, -3 * T:]), ref[:, -3 * T:], TOL_IIR_F32, "tail S=%d tiles=%d" % (S, tiles))
    assert np.max(np.abs(_cpu(so) - rs)) <= TOL_IIR_F32 * 0.1
    head = O.sos(_cpu(x[:, :4 * T]), sec, state_in=s0)
    assert_close(_cpu(y[:, :4 * T]), head, TOL_IIR_F32, "head S=%d tiles=%d" % (S, tiles))
