"""Calls whose tiles, carries and transforms take several forms: what one form
leaves in a workspace is nothing to the next, and each form gives all the
outputs of the call.  Against the FP64 oracle, or the scan."""
import numpy as np
import pytest
import torch

import paper_2504_08624_amd as tfx
from paper_2504_08624_amd import design, lib, signals
from oracle import oracle as O
from tests.metrics import TOL_IIR_F32, assert_close

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


def _peaks(S, q):
    """Peaking sections from 4 kHz up; q = 400 puts every pole where the carry is FP64."""
    return np.concatenate([design.peaking(f, q, 6.0, 48000.0) for f in np.linspace(4000.0, 15000.0, S)]
                          ).astype(np.float32)


@pytest.mark.parametrize("S,C,blocks", [
    pytest.param(3, 2, (300_000, 100_000, 300_000, 20_000, 512, 100_000), id="one pass over 64 workgroups, one under"),
    pytest.param(8, 64, (64 * T, 2 * T, 2 * T, 64 * T, 2 * T), id="last tile apart, all tiles together"),
])
def test_fp64_carries_over_blocks_of_every_form(S, C, blocks):
    """A stream whose blocks take turns between the forms: no block may take a
    record that another block left."""
    x = _x(C, sum(blocks), (951, S))
    sec = _peaks(S, 400.0)
    want, regs = O.sos(x, sec, return_state=True)
    st = tfx.ChainStream([("sos", _gpu(sec))], C, max(blocks))
    n0, out = 0, []
    for b in blocks:
        out.append(_cpu(st.process(_gpu(x[:, n0:n0 + b]))))
        n0 += b
        assert_close(out[-1], want[:, n0 - b:n0], TOL_IIR_F32, "block of %d up to %d" % (b, n0))
    assert np.max(np.abs(_cpu(st._state[st._cur]) - regs)) <= TOL_IIR_F32 * np.max(np.abs(regs)), "registers"


@pytest.mark.parametrize("hiq", [False, True])
@pytest.mark.parametrize("S", [1, 6, 8, 9])
@pytest.mark.parametrize("C,N", [(3, 1), (3, 512), (3, T), (200, 700)])
def test_checkpoint_and_registers_of_one_tile(C, N, S, hiq):
    """tfx_sos with registers and checkpoints: a tile that is alone enters with
    the given registers, and its checkpoint says so (the output buffer starts
    filled with something else)."""
    x = _gpu(_x(C, N, (952, S, N)))
    sec = _gpu(_peaks(S, 400.0 if hiq else 1.0))
    s0 = _gpu((0.05 * signals.rng(953, S, N).standard_normal((C, S, 2))).astype(np.float32))
    nb = lib.size_out()
    lib.call("tfx_sos_workspace_size", C, N, S, nb)
    ws = torch.empty(nb.value, dtype=torch.uint8, device=DEV)
    for si in (s0, None):
        y, so = torch.empty_like(x), torch.empty_like(s0)
        ck = torch.full((C, 1, S, 2), 7.0, device=DEV)
        lib.call("tfx_sos", x.data_ptr(), y.data_ptr(), C, N, N, N, sec.data_ptr(), S,
                 si.data_ptr() if si is not None else None, so.data_ptr(), ck.data_ptr(), ws.data_ptr(), nb.value,
                 torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(ck[:, 0], torch.zeros_like(s0) if si is None else si)


def test_inverse_stft_of_no_samples():
    """One centred frame has no output: nothing is fetched or looked at, and what was
    refused still is."""
    spec = torch.randn(2, 513, 1, dtype=torch.complex64, device=DEV)
    for w in (None, torch.ones(1024, device=DEV), torch.zeros(1024, device=DEV)):
        assert tuple(tfx.istft(spec, 1024, 256, window=w).shape) == (2, 0)
    with pytest.raises(ValueError):
        tfx.istft(spec, 1024, 256, window=torch.ones(1000, device=DEV))
    with pytest.raises(ValueError):                          # the window's sum vanishes inside the output
        tfx.istft(torch.randn(2, 513, 9, dtype=torch.complex64, device=DEV), 1024, 256,
                  window=torch.zeros(1024, device=DEV))


@pytest.mark.parametrize("taps", [0, 201])
def test_low_frequency_stream_of_mixed_blocks(taps):
    """Slow registers (peaks from 250 Hz) through blocks of one tile and of several."""
    C, sizes = 3, (512, 4 * T + 3, 512, 1, 2 * T, 700, 230_000, 512)
    x = _x(C, sum(sizes), (954, taps))
    sec = np.concatenate([design.peaking(f, 1.0, 6.0, 48000.0) for f in (250.0, 700.0, 2000.0)]).astype(np.float32)
    stages = [("sos", sec)]
    if taps:
        stages.insert(0, ("fir", design.fir_lowpass(taps, 9000.0, 48000.0).astype(np.float32)))
    st = tfx.ChainStream([(k, _gpu(c)) for k, c in stages], C, max(sizes))
    ends = np.cumsum(sizes)
    out = [_cpu(st.process(_gpu(x[:, e - b:e]))) for e, b in zip(ends, sizes)]
    assert_close(np.concatenate(out, axis=1), O.chain(x, stages), TOL_IIR_F32, "taps %d" % taps)
