"""The filtering work that users of this framework have it do, one case each.

A case names a kind of call, its sizes and its filters:

  chain   tfx.chain on a [C, N] signal: a low-pass FIR and an equaliser of
          second-order sections, coefficients resident on the device
  fir     tfx.fir alone (short, medium and long filters; fp32 and matrix-core
          operand types)
  sos     tfx.sos with registers carried in and out (one part of a long file)
  batch   tfx.sos_batched: clips of different lengths, each its own cascade
  stream  ChainStream.process: consecutive short blocks of a live stream
  train   tfx.chain under autograd: output, input gradient and the gradients
          of taps and sections for a given upstream gradient (a trainable
          filter inside a larger model)
  stft    tfx.stft with a device-resident window
  istft   tfx.istft of such a spectrum

Signals are white noise of standard deviation 0.1, 1/f noise with an
exponential sweep, or noise with a decaying envelope, as the repository's
benchmark workloads draw them, made on the device from the seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2504_08624_amd as tfx

FS = 48_000.0
DEV = "cuda:0"

# ------------------------------------------------------------------ the cases


def listed():
    return [
        # a live stream of 512-sample blocks through the benchmark's chain: latency per block counts
        {"name": "stream_512", "kind": "stream", "C": 8, "N": 512, "blocks": 4, "taps": 1023, "S": 6, "f": 250.0},
        # a ten-second stereo clip through a short FIR and an equaliser: launch-bound
        {"name": "chain_short", "kind": "chain", "C": 2, "N": 480_000, "taps": 101, "S": 2, "f": 1_000.0,
         "compute": "f32", "signal": "white"},
        # the benchmark's headline: two minutes of 8 channels, 1023 taps and 6 sections
        {"name": "chain_mid", "kind": "chain", "C": 8, "N": 5_760_000, "taps": 1023, "S": 6, "f": 250.0,
         "compute": "f32", "signal": "pink"},
        # the same chain with bf16 FIR operands, at an odd length
        {"name": "chain_bf16", "kind": "chain", "C": 8, "N": 5_292_001, "taps": 1023, "S": 6, "f": 250.0,
         "compute": "bf16", "signal": "pink"},
        # one minute of 64 channels at 96 kHz through an 8191-tap low-pass
        {"name": "fir_long", "kind": "fir", "C": 64, "N": 5_760_000, "taps": 8191, "compute": "f32",
         "signal": "white"},
        # the paper's largest channel count, two minutes at 44.1 kHz less a sample (rows of odd length)
        {"name": "iir_multi", "kind": "sos", "C": 12, "N": 5_291_999, "S": 4, "rlo": 0.5, "rhi": 0.95,
         "signal": "white"},
        # thirty stereo seconds through resonators close to the unit circle (FP64 carry)
        {"name": "high_q", "kind": "sos", "C": 2, "N": 1_440_000, "S": 6, "rlo": 0.999, "rhi": 0.99995,
         "signal": "white"},
        # a data-augmentation batch: 48 clips of 1 to 30 s at 44.1 kHz, 1 to 16 channels, 1 to 6 sections
        {"name": "ragged_48", "kind": "batch", "clips": 48, "nmin": 44_100, "nmax": 1_323_000, "cmax": 16, "smax": 6,
         "rhi": 0.999, "mix": 4},
        # a trainable filter in a model: 32 stereo items of 4 s, 255 taps and 8 biquads
        {"name": "train_items", "kind": "train", "C": 64, "N": 192_000, "taps": 255, "S": 8, "f": 1_000.0,
         "signal": "white"},
        # forward and backward of the headline chain
        {"name": "train_mid", "kind": "train", "C": 8, "N": 5_760_000, "taps": 1023, "S": 6, "f": 250.0,
         "signal": "pink"},
        # spectrogram of the headline signal
        {"name": "stft_2048", "kind": "stft", "C": 8, "N": 5_760_000, "n_fft": 2048, "hop": 512},
        # and its resynthesis
        {"name": "istft_2048", "kind": "istft", "C": 8, "N": 5_760_000, "n_fft": 2048, "hop": 512},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, channels, lo, hi, most):
    """C of `channels` and N log-uniform in [lo, hi] with C * N <= most; odd as often as even."""
    C = rng.choice(channels)
    return C, _log(rng, lo, max(lo + 1, min(hi, most // C)))


def draw(rng):
    kind = rng.choice(["chain", "chain", "train", "train", "fir", "fir", "sos", "sos", "batch", "stream", "stft",
                       "istft"])
    c = {"kind": kind}
    sig = rng.choice(["white", "pink", "decay"])
    if kind == "chain":
        c["C"], c["N"] = _shape(rng, [1, 2, 3, 6, 8, 12, 16], 20_000, 8_000_000, 50_000_000)
        c.update(taps=_log(rng, 16, 2049), S=rng.randint(1, 8), f=round(math.exp(rng.uniform(5.86, 8.0)), 1),
                 compute=rng.choice(["f32", "f32", "f32", "bf16", "f16"]), signal=sig)
    elif kind == "train":
        c["C"], c["N"] = _shape(rng, [1, 2, 8, 31, 64], 20_000, 5_760_000, 46_080_000)
        c.update(taps=_log(rng, 32, 1025), S=rng.randint(1, 8), f=round(math.exp(rng.uniform(5.86, 8.0)), 1),
                 signal=sig)
    elif kind == "fir":
        c["C"], c["N"] = _shape(rng, [1, 2, 5, 8, 12, 64], 20_000, 8_000_000, 100_000_000)
        c["compute"] = rng.choice(["f32", "f32", "f32", "bf16", "f16", "bf16x3"])
        c["taps"] = _log(rng, 8, 8193 if c["compute"] == "f32" else 2049)
        c["signal"] = sig
    elif kind == "sos":
        c["C"], c["N"] = _shape(rng, [1, 2, 3, 6, 8, 12], 20_000, 8_000_000, 64_000_000)
        highq = rng.random() < 0.25
        c.update(S=rng.randint(1, 8), rlo=0.999 if highq else 0.3, rhi=0.9999 if highq else 0.97, signal=sig)
    elif kind == "batch":
        c.update(clips=rng.randint(3, 60), nmin=_log(rng, 5_000, 50_000), nmax=_log(rng, 60_000, 800_000),
                 cmax=rng.choice([1, 2, 8, 16]), smax=rng.randint(1, 6), rhi=rng.choice([0.95, 0.99, 0.999]),
                 mix=rng.randint(0, 10_000))
    elif kind == "stream":
        c.update(C=rng.choice([1, 2, 8, 12]), N=_log(rng, 64, 4096), blocks=rng.choice([2, 4]),
                 taps=_log(rng, 32, 1025), S=rng.randint(1, 6), f=round(math.exp(rng.uniform(5.86, 8.0)), 1))
    else:
        n = rng.choice([256, 512, 1024, 2048, 4096])
        c["C"], c["N"] = _shape(rng, [1, 2, 8], 50_000, 5_760_000, 40_000_000)
        c.update(n_fft=n, hop=n // rng.choice([2, 4]))
    return c


# ------------------------------------------------------------------ signals and filters


def _gen(seed, *key):
    g = torch.Generator(device=DEV)
    k = int(seed)
    for v in key:
        k = (k * 1_000_003 + int(v) + 1) % (1 << 62)
    g.manual_seed(k)
    return g


def _signal(kind, C, N, seed):
    x = torch.empty((C, N), dtype=torch.float32, device=DEV)
    t = torch.arange(N, dtype=torch.float64, device=DEV)
    if kind == "pink":                     # 1/f noise (RMS 0.1) and a 20 Hz - 20 kHz sweep
        k = math.log(1000.0)
        sweep = (0.5 * torch.sin(2 * math.pi * 20.0 * N / FS / k * (torch.exp(t * (k / N)) - 1.0))).float()
        n2 = 1 << max(1, (N - 1).bit_length())
        f = torch.arange(n2 // 2 + 1, dtype=torch.float32, device=DEV)
        shape = torch.where(f > 0, f.clamp(min=1).rsqrt(), torch.zeros_like(f))
    for c in range(C):
        w = torch.randn(N, generator=_gen(seed, c), dtype=torch.float32, device=DEV)
        if kind == "pink":
            p = torch.fft.irfft(torch.fft.rfft(w, n2) * shape, n2)[:N]
            x[c] = p * (0.1 / p.square().mean().sqrt()) + sweep
        elif kind == "decay":              # struck notes: a decaying envelope every second or so
            x[c] = 0.3 * w * torch.exp(-(t % 50_000) / 9_000.0).float()
        else:
            x[c] = 0.1 * w
    return x


def _lowpass(M, fc):
    """Hamming windowed sinc, unit gain at DC."""
    n = np.arange(M) - (M - 1) / 2.0
    w = 2.0 * fc / FS
    h = w * np.sinc(w * n) * (0.54 + 0.46 * np.cos(2.0 * np.pi * n / max(M - 1, 1)))
    return (h / h.sum()).astype(np.float32)


def _equaliser(S, f):
    """Half the sections a 12 kHz Butterworth low-pass, the rest peaking filters from f upwards (alternating
    boost and cut), textbook biquads [b0 b1 b2 a1 a2]."""
    rows = []                              # b0 b1 b2 a1 a2 a0
    for i in range(S // 2):
        w0 = 2.0 * np.pi * 12_000.0 / FS
        q = 1.0 / (2.0 * np.cos(np.pi * (2 * i + 1) / (4 * (S // 2))))
        al, c = np.sin(w0) / (2.0 * q), np.cos(w0)
        rows.append([(1 - c) / 2, 1 - c, (1 - c) / 2, -2 * c, 1 - al, 1 + al])
    for i in range(S - S // 2):
        w0 = 2.0 * np.pi * min(f * 2.7 ** i, 16_000.0) / FS
        A = 10.0 ** ((6.0 if i % 2 == 0 else -9.0) / 40.0)
        al, c = np.sin(w0) / (2.0 * (0.8 + 0.6 * i)), np.cos(w0)
        rows.append([1 + al * A, -2 * c, 1 - al * A, -2 * c, 1 - al / A, 1 + al / A])
    r = np.asarray(rows)
    return np.ascontiguousarray(r[:, :5] / r[:, 5:]).astype(np.float32)


def _resonators(rng, S, rlo, rhi):
    """Random sections: poles r exp(+-i th) of radius [rlo, rhi], zeros on the unit circle, unit gain at the pole angle."""
    rows = []
    for _ in range(S):
        r, th, tz = rng.uniform(rlo, rhi), rng.uniform(0.05, 0.95) * np.pi, rng.uniform(0.0, 1.0) * np.pi
        b, a = np.array([1.0, -2 * np.cos(tz), 1.0]), np.array([1.0, -2 * r * np.cos(th), r * r])
        z = np.exp(-1j * th * np.arange(3))
        g = max(abs((b * z).sum() / (a * z).sum()), 1e-3)
        rows.append(np.concatenate([b / g, a[1:]]))
    return np.asarray(rows, dtype=np.float32).reshape(S, 5)


def _cutoff(case):
    return 6_000.0 if case["taps"] > 200 else 10_000.0


def _clips(case, seed):
    rng = np.random.default_rng([11, case["mix"]])
    out = []
    for i in range(case["clips"]):
        N = int(rng.integers(case["nmin"], case["nmax"] + 1))
        C = int(rng.integers(1, case["cmax"] + 1))
        sec = _resonators(rng, int(rng.integers(1, case["smax"] + 1)), 0.5, case["rhi"])
        x = torch.randn((C, N), generator=_gen(seed, i), dtype=torch.float32, device=DEV).mul_(0.1)
        out.append((x, sec))
    return out


def _parts(case, seed):
    """Inputs and coefficients of a case (float32: arrays for filters, device tensors for signals)."""
    k = case["kind"]
    if k == "batch":
        return {"clips": _clips(case, seed)}
    p = {}
    if k == "stream":
        p["x"] = _signal("white", case["C"], case["N"] * case["blocks"], seed)
    else:
        p["x"] = _signal(case.get("signal", "pink"), case["C"], case["N"], seed)
    if "taps" in case:
        p["h"] = _lowpass(case["taps"], _cutoff(case))
    if k == "sos":
        p["s"] = _resonators(np.random.default_rng([12, case["S"]]), case["S"], case["rlo"], case["rhi"])
        p["s0"] = 0.05 * torch.randn((case["C"], case["S"], 2), generator=_gen(seed, 777), dtype=torch.float32,
                                     device=DEV)
    elif "S" in case:
        p["s"] = _equaliser(case["S"], case["f"])
    if k == "train":
        p["g"] = _residual(case, p, seed)
    if k in ("stft", "istft"):
        p["w"] = torch.hann_window(case["n_fft"], dtype=torch.float32, device=DEV)
    return p


def _residual(case, p, seed):
    """Upstream gradient of a squared error: the output less that of the same chain tuned elsewhere, and some noise."""
    N = case["N"]
    n = _fft_len(N + case["taps"] + 4096)
    f64 = lambda a: torch.from_numpy(a).to(DEV).double()  # noqa: E731
    h = f64(p["h"])
    D = _response(h, f64(p["s"]), n) - _response(h, f64(_equaliser(case["S"], 1.3 * case["f"])), n)
    g = torch.randn((case["C"], N), generator=_gen(seed, 778), dtype=torch.float32, device=DEV).mul_(0.01)
    for c in range(case["C"]):
        g[c] += torch.fft.irfft(torch.fft.rfft(p["x"][c].double(), n) * D, n)[:N].float()
    return g


# ------------------------------------------------------------------ prepare / run


def prepare(case, seed):
    p = _parts(case, seed)
    k = case["kind"]
    s = {"case": dict(case)}
    if k == "batch":
        s["xs"] = [x for x, _ in p["clips"]]
        s["secs"] = [torch.from_numpy(c).to(DEV) for _, c in p["clips"]]
        return s
    s["x"] = p["x"]
    if "h" in p:
        s["h"] = torch.from_numpy(p["h"]).to(DEV)
    if "s" in p:
        s["s"] = torch.from_numpy(p["s"]).to(DEV)
    if k == "sos":
        s["s0"] = p["s0"]
    if k == "train":
        s["g"] = p["g"]
        for n in ("x", "h", "s"):
            s[n].requires_grad_(True)
    if k == "stream":
        s["blocks"] = [b.contiguous() for b in p["x"].split(case["N"], dim=1)]
        s["stream"] = tfx.ChainStream([("fir", s["h"]), ("sos", s["s"])], channels=case["C"], max_block=case["N"],
                                      device=DEV)
    if k in ("stft", "istft"):
        s["w"] = p["w"]
    if k == "istft":
        s["spec"] = _spectrum(s["x"], case, s["w"])
        s["x"] = None
    return s


def _spectrum(x, case, w):
    """The frames of x as a mixing program holds them (frame-major storage, [C, F, T] view)."""
    X = torch.stft(x, case["n_fft"], case["hop"], window=w, center=True, return_complex=True)
    return X.transpose(1, 2).contiguous().transpose(1, 2)


def run(state):
    c = state["case"]
    k = c["kind"]
    if k == "chain":
        return tfx.chain(state["x"], [("fir", state["h"]), ("sos", state["s"])], compute=c["compute"])
    if k == "fir":
        return tfx.fir(state["x"], state["h"], compute=c["compute"])
    if k == "sos":
        return tfx.sos(state["x"], state["s"], state_in=state["s0"], return_state=True)
    if k == "batch":
        return tfx.sos_batched(state["xs"], state["secs"])
    if k == "stream":
        return [state["stream"].process(b) for b in state["blocks"]]
    if k == "train":
        y = tfx.chain(state["x"], [("fir", state["h"]), ("sos", state["s"])])
        gx, gh, gs = torch.autograd.grad(y, (state["x"], state["h"], state["s"]), state["g"])
        return {"y": y, "gx": gx, "gh": gh, "gs": gs}
    if k == "stft":
        return tfx.stft(state["x"], c["n_fft"], c["hop"], window=state["w"])
    return tfx.istft(state["spec"], c["n_fft"], c["hop"], window=state["w"],
                     length=c["N"] // c["hop"] * c["hop"])


# ------------------------------------------------------------------ the least work


def _fir_flops(M):
    """Operations per output of an M-tap convolution: the direct sum, or overlap-save transforms of 8 M points."""
    return float(min(2 * M, 2 * 5 * 8 / 7 * math.log2(8 * max(M, 2)) / 2 + 8))


def work(case):
    k = case["kind"]
    if k == "batch":
        rng = np.random.default_rng([11, case["mix"]])
        n = f = 0
        for _ in range(case["clips"]):
            N = int(rng.integers(case["nmin"], case["nmax"] + 1))
            C = int(rng.integers(1, case["cmax"] + 1))
            S = int(rng.integers(1, case["smax"] + 1))
            for _ in range(S):
                rng.uniform(), rng.uniform(), rng.uniform()
            n += C * N
            f += C * N * 9 * S
        return {"bytes": 8.0 * n, "flops": float(f)}
    n = float(case["C"]) * case["N"] * case.get("blocks", 1)
    if k in ("stft", "istft"):
        nf = case["n_fft"]
        frames = case["C"] * (case["N"] // case["hop"] + 1)
        return {"bytes": 4 * n + 8.0 * frames * (nf // 2 + 1), "flops": frames * (2.5 * nf * math.log2(nf) + 2 * nf)}
    f = (_fir_flops(case["taps"]) if "taps" in case else 0.0) + 9.0 * case.get("S", 0)
    if k == "train":
        # x read, y written; the upstream gradient and x read, the input gradient written
        return {"bytes": 20 * n, "flops": 3 * f * n}
    return {"bytes": 8 * n, "flops": f * n}


# ------------------------------------------------------------------ the same in 64 bits


def _fft_len(n):
    best = 1 << max(1, (n - 1).bit_length())
    for m in (3, 5, 9, 15):
        v = m << max(1, (-(-n // m) - 1).bit_length())
        if n <= v < best:
            best = v
    return best


def _ring(sec):
    """Samples after which the cascade's response is below 64-bit rounding."""
    r = 0.0
    for b0, b1, b2, a1, a2 in np.asarray(sec, dtype=np.float64):
        r = max([r] + [abs(z) for z in np.roots([1.0, a1, a2])])
    return 64 if r < 1e-3 else int(46.0 / -math.log(r)) + 64 * (len(sec) + 1)


def _z(n):
    w = torch.arange(n // 2 + 1, dtype=torch.float64, device=DEV) * (-2.0 * math.pi / n)
    return torch.polar(torch.ones_like(w), w)


def _response(h, s, n):
    """H on the n-point grid, differentiable in h and s (float64 device tensors or None)."""
    H = torch.fft.rfft(h, n) if h is not None else None
    if s is not None:
        z = _z(n)
        for row in s:
            S = (row[0] + z * (row[1] + z * row[2])) / (1.0 + z * (row[3] + z * row[4]))
            H = S if H is None else H * S
    return H


def _filter(x, H, n):
    """Row by row, so that long signals fit."""
    N = x.shape[-1]
    return torch.stack([torch.fft.irfft(torch.fft.rfft(r, n) * H, n)[:N] for r in x])


def _quantised(t, compute):
    if compute == "bf16":
        return t.to(torch.bfloat16).double()
    if compute == "f16":
        return t.to(torch.float16).double()
    return t.double()


def _sos_exact(x, s, s0):
    """Zero-state response plus the registers' decay, and the registers after the last sample."""
    C, N = x.shape
    n = _fft_len(N + _ring(s.cpu().numpy()))
    z = _z(n)
    ys, ends = [], []
    for c in range(C):
        y, end = x[c].double(), []
        Y = torch.fft.rfft(y, n)
        for i, row in enumerate(s):
            A = 1.0 + z * (row[3] + z * row[4])
            last = y[-2:]
            Y = ((row[0] + z * (row[1] + z * row[2])) * Y + (s0[c, i, 0] + z * s0[c, i, 1])) / A
            y = torch.fft.irfft(Y, n)[:N]
            # the filtered row is cut at N before the next section, as only its first N samples are heard
            Y = torch.fft.rfft(y, n)
            s2b = row[2] * last[0] - row[4] * y[-2]
            end.append(torch.stack([row[1] * last[1] - row[3] * y[-1] + s2b, row[2] * last[1] - row[4] * y[-1]]))
        ys.append(y)
        ends.append(torch.stack(end))
    return torch.stack(ys), torch.stack(ends)


def exact(case, seed):
    k = case["kind"]
    p = _parts(case, seed)
    dev = lambda a: torch.from_numpy(a).to(DEV).double()  # noqa: E731
    if k == "batch":
        out = []
        for x, sec in p["clips"]:
            n = _fft_len(x.shape[1] + _ring(sec))
            out.append(_filter(x.double(), _response(None, dev(sec), n), n))
        return out
    if k in ("chain", "fir"):
        # bf16 and f16 round the FIR's operands: their exact result is that of the rounded operands
        h = _quantised(torch.from_numpy(p["h"]).to(DEV), case["compute"])
        s = dev(p["s"]) if "s" in p else None
        n = _fft_len(case["N"] + case["taps"] + (_ring(p["s"]) if s is not None else 0))
        H = _response(h, s, n)
        N = case["N"]
        return torch.stack([torch.fft.irfft(torch.fft.rfft(_quantised(r, case["compute"]), n) * H, n)[:N]
                            for r in p["x"]])
    if k == "sos":
        return _sos_exact(p["x"], dev(p["s"]), p["s0"].double())
    if k == "stream":
        n = _fft_len(p["x"].shape[1] + case["taps"] + _ring(p["s"]))
        y = _filter(p["x"].double(), _response(dev(p["h"]), dev(p["s"]), n), n)
        return list(y.split(case["N"], dim=1))
    if k == "train":
        h, s = dev(p["h"]).requires_grad_(True), dev(p["s"]).requires_grad_(True)
        N = case["N"]
        n = _fft_len(N + case["taps"] + _ring(p["s"]))
        ys, gxs, gh, gs = [], [], 0, 0
        for r, g in zip(p["x"], p["g"]):
            xr = r.detach().double().requires_grad_(True)
            y = torch.fft.irfft(torch.fft.rfft(xr, n) * _response(h, s, n), n)[:N]
            a, b, c = torch.autograd.grad(y, (xr, h, s), g.double())
            ys.append(y.detach())
            gxs.append(a)
            gh, gs = gh + b, gs + c
        return {"y": torch.stack(ys), "gx": torch.stack(gxs), "gh": gh, "gs": gs}
    w = p["w"].double()
    if k == "stft":
        return torch.stft(p["x"].double(), case["n_fft"], case["hop"], window=w, center=True, return_complex=True)
    spec = _spectrum(p["x"], case, p["w"])
    return torch.istft(spec.to(torch.complex128), case["n_fft"], case["hop"], window=w, center=True,
                       length=case["N"] // case["hop"] * case["hop"])
