"""Throughput of the multichannel FIR -> IIR-SOS chain on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--quick] [--no-cpu-baseline]

Headline workload (the mid-size chain): 8 channels x 5,760,000 samples
(120 s at 48 kHz), fp32, per-channel seeded 1/f noise plus a 20 Hz-20 kHz log
sweep; chain = 1023-tap Hamming band-pass FIR | 8th-order Chebyshev-I
low-pass (4 sections) | 2 peaking EQs: one FIR plus a 6-section cascade.

A step is one full tfx_chain call on the resident input: the device table
build (tfx_chain_prepare) followed by the fused filter kernel
(tfx_chain_run).  W untimed steps, then K timed steps between two device
synchronisations; `value` is channel-samples per second of the whole step.
HIP events recorded on the launch stream around every tfx_chain_run give the
filter kernel's average duration for the roofline (algorithmic bytes = 8 B
per channel-sample: read x once, write y once; the bracket also holds the
launches of the scan behind the block kernel, which exit at once); events around every step
give its median and spread, ten more steps run "cold" (512 MB written before
each, more than the last-level cache holds), and a plain device copy of the
input gives the achievable bandwidth the HBM figure is also quoted against.  The same loop is then timed
for forward + backward (forward with tile checkpoints, then the adjoint of
the chain for a fixed upstream gradient: gradients of input, taps and
sections).

Unless --quick, the other workloads are measured once each (context, in
"secondary"): the short chain (also at the headline's size), the 8191-tap
FIR by FFT (fp32) and by the matrix-core Toeplitz product (bf16, fp16, split
bf16), the headline's 1023-tap FIR alone in every form, the ragged batch of
256 clips (autotuned, one hipGraph replay, against one tfx_sos call per
clip), the differentiable workload's forward and forward + backward, the
Wave pipe, streaming blocks, and the STFT / inverse STFT of the headline
signal.  Errors are measured against the oracle on sampled outputs.
`--leg NAME` runs one of these alone (for kernel profiles).

The CPU baseline runs the FP64 oracle (test infrastructure: plain C, one
OpenMP thread per channel) on a bounded sample of the headline input and
reports its throughput.  Prints one JSON line.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0        # MI355X published HBM3E bandwidth
MFMA_BF16_PEAK_TFS = 2500.0  # dense bf16 / fp16 matrix peak
# fp32 vector peak without packed-FP32 instructions (disabled at build time):
# 256 CU x 4 SIMD x 16 lanes x 2 flop x 2.4 GHz
VALU_F32_PEAK_TFS = 78.6


def chain_flops_per_sample(C, N, V):
    """Vector-unit flops per channel-sample of the short-memory form of the
    chain (FIR and cascade as one FIR on 16384-point blocks): one forward and one
    inverse complex transform (5 n log2 n each) and a spectrum product (6 a bin)
    per block, two tiles of 16384 - V samples of a channel, V the chain's memory
    (None: the chain ran as a scan)."""
    if not V:
        return None
    n = 16384
    blocks = C * -(-(-(-N // (n - V))) // 2)
    return blocks * (2 * 5 * n * 14 + 6 * n) / (C * N)


def measured_traffic():
    """HBM bytes per launch of the chain's block kernel from the committed
    rocprofv3 counter runs (profiles/chain_mid_traffic.json), or None when the
    kernel's sources have changed since the counters were taken."""
    import hashlib
    path = os.path.join(ROOT, "profiles", "chain_mid_traffic.json")
    try:
        rec = json.load(open(path))
        h = hashlib.sha256()
        for f in rec["sources"]:
            h.update(open(os.path.join(ROOT, f), "rb").read())
    except (OSError, ValueError, KeyError):
        return None
    return rec["traffic_bytes_per_launch"] if h.hexdigest() == rec["sources_sha256"] else None


def cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--quick", action="store_true", help="headline workload only")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--stft-only", action="store_true", help="only the STFT leg (for kernel profiles)")
    ap.add_argument("--leg", action="append", choices=LEGS,
                    help="run only this context leg (repeatable; for kernel profiles); no headline")
    ap.add_argument("--copy-probe", action="store_true",
                    help="accepted for older profile commands; the device copy of the input is always timed")
    return ap.parse_args()


def log(msg):
    print("bench: " + msg, file=sys.stderr, flush=True)


def rel_err(y, ref):
    num = np.linalg.norm(np.asarray(y, np.float64) - ref, axis=-1)
    den = np.linalg.norm(ref, axis=-1)
    return float((num / np.where(den > 0, den, 1.0)).max())


def timed(torch, fn, reps, stream):
    for _ in range(2):
        fn()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        fn()
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) / reps


LEGS = ("chain_short", "fir_long", "fir_mid_forms", "ragged", "chain_short_large", "learnable", "wave_pipe",
        "chain_mid_compute", "stream", "stft")


def secondary(torch, dev, stream, only=None):
    """The context legs; `only`: a set of leg names (None = all)."""
    import paper_2504_08624_amd as tfx
    from oracle import oracle as O
    from paper_2504_08624_amd import workloads
    out = {}

    def want(name):
        return only is None or name in only

    if want("chain_short"):
        log("chain_short")
        w = workloads.chain_short()
        x = torch.from_numpy(w.x).to(dev)
        st = [(k, torch.from_numpy(c).to(dev)) for k, c in w.stages]
        s = timed(torch, lambda: tfx.chain(x, st), 20, stream)
        y = tfx.chain(x, st).cpu().numpy()
        out["chain_short"] = {"workload": "2 x 480,000, 101-tap FIR | Butterworth HP (2 SOS)",
                              "Msamples_per_s": round(x.numel() / s / 1e6, 1), "ms": round(s * 1e3, 4),
                              "rel_err": rel_err(y, O.chain(w.x, w.stages)), "tolerance": 1e-4}
        del x, st

    if want("fir_long"):
        log("fir_long")
        w = workloads.fir_long()
        x = torch.from_numpy(w.x).to(dev)
        h = torch.from_numpy(w.stages[0][1]).to(dev)
        n = x.numel()
        M = h.numel()
        pos = np.linspace(0, w.x.shape[1] - 1, 257).astype(np.int64)
        chans = [0, 21, 63]
        ref = O.fir_at(w.x[chans], w.stages[0][1], pos)
        o_sec = O.last_seconds()
        res = {"workload": "64 x 5,760,000, 8191-tap low-pass", "error": "rel RMS on 3 ch x 257 sampled outputs",
               "oracle": {"Msamples_per_s": round(len(chans) * pos.size / o_sec / 1e6, 4),
                          "cores": min(len(chans), O.threads()),
                          "sample": "3 ch x 257 outputs by direct convolution, steady clock around the C loop"}}
        for name, kw, tol in [("fft_f32", {}, 1e-5), ("fft4096_parts_f32", {"algo": "fft"}, 1e-5),
                              ("toeplitz_bf16", {"compute": "bf16"}, 1e-2),
                              ("toeplitz_f16", {"compute": "f16"}, 1e-2), ("toeplitz_bf16x3", {"compute": "bf16x3"}, None)]:
            s = timed(torch, lambda: tfx.fir(x, h, **kw), 3, stream)
            yy = tfx.fir(x, h, **kw)[chans][:, pos].cpu().numpy()
            e = {"Msamples_per_s": round(n / s / 1e6, 1), "ms": round(s * 1e3, 3), "rel_err": rel_err(yy, ref)}
            if tol:
                e["tolerance"] = tol
            if name.startswith("toeplitz"):
                flops = 2.0 * n * M * (3 if name.endswith("x3") else 1)
                e["mfma_TFLOP_per_s"] = round(flops / s / 1e12, 1)
                e["mfma_frac"] = round(flops / s / 1e12 / MFMA_BF16_PEAK_TFS, 4)
            res[name] = e
        out["fir_long"] = res
        del x, h

    if want("fir_mid_forms"):
        log("fir_mid_forms")
        w = workloads.chain_mid()
        x = torch.from_numpy(w.x).to(dev)
        h = torch.from_numpy(w.stages[0][1]).to(dev)
        n = x.numel()
        M = h.numel()
        pos = np.linspace(0, w.x.shape[1] - 1, 513).astype(np.int64)
        chans = [0, 5]
        ref = O.fir_at(w.x[chans], w.stages[0][1], pos)
        res = {"workload": "chain_mid's 1023-tap band-pass FIR alone on its signal (8 x 5,760,000)",
               "error": "rel RMS on 2 ch x 513 sampled outputs"}
        for name, kw, tol, reps in [("direct_f32", {"algo": "direct"}, 1e-5, 3), ("fft_f32", {"algo": "fft"}, 1e-5, 10),
                                    ("fft16k_f32", {"algo": "fft16k"}, 1e-5, 10),
                                    ("toeplitz_bf16", {"compute": "bf16"}, 1e-2, 10),
                                    ("toeplitz_f16", {"compute": "f16"}, 1e-2, 10),
                                    ("toeplitz_bf16x3", {"compute": "bf16x3"}, 1e-4, 10)]:
            s = timed(torch, lambda: tfx.fir(x, h, **kw), reps, stream)
            yy = tfx.fir(x, h, **kw)[chans][:, pos].cpu().numpy()
            e = {"ms": round(s * 1e3, 4), "Msamples_per_s": round(n / s / 1e6, 1), "rel_err": rel_err(yy, ref),
                 "tolerance": tol}
            if name.startswith("toeplitz"):
                flops = 2.0 * n * M * (3 if name.endswith("x3") else 1)
                e["mfma_TFLOP_per_s"] = round(flops / s / 1e12, 1)
            res[name] = e
        out["fir_mid_forms"] = res
        del x, h

    if want("ragged"):
        log("ragged batch")
        clips = workloads.ragged()
        xs = [torch.from_numpy(c[0]).to(dev) for c in clips]
        ss = [torch.from_numpy(c[1]).to(dev) for c in clips]
        n = sum(t.numel() for t in xs)
        b = tfx.SosBatch(xs, ss)
        cfg, _ = b.tune(reps=2)
        s_b = timed(torch, b.run, 5, stream)
        # the batch as one captured graph (one hipGraphLaunch per replay)
        gs = torch.cuda.Stream()
        gs.wait_stream(stream)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(gs):
            with torch.cuda.graph(graph, stream=gs):
                b.run()
        stream.wait_stream(gs)
        s_g = timed(torch, graph.replay, 10, stream)
        s_l = timed(torch, lambda: [tfx.sos(a, c) for a, c in zip(xs, ss)], 3, stream)
        graph.replay()
        ys = b.ys
        errs = [rel_err(ys[i].cpu().numpy(), O.sos(clips[i][0], clips[i][1])) for i in (0, 97, 201)]
        c0 = time.perf_counter()
        c_sec = 0.0
        c_n = 0
        for i in (0, 97, 201):
            O.sos(clips[i][0], clips[i][1])
            c_sec += O.last_seconds()
            c_n += clips[i][0].size
        out["ragged_batch"] = {"workload": "256 clips @44.1 kHz, 1-30 s, 1-16 ch, 1-6 SOS each",
                               "samples": n, "tuned": cfg, "Msamples_per_s": round(n / s_g / 1e6, 1),
                               "ms": round(s_g * 1e3, 3), "timing": "one hipGraph replay of the batched run",
                               "eager_run_ms": round(s_b * 1e3, 3),
                               "hbm_frac": round(8.0 * n / s_g / 1e9 / HBM_PEAK_GBS, 4),
                               "per_clip_calls_ms": round(s_l * 1e3, 3),
                               "speedup_vs_per_clip": round(s_l / s_g, 2), "rel_err_3_clips": max(errs),
                               "tolerance": 1e-4,
                               "oracle": {"Msamples_per_s": round(c_n / c_sec / 1e6, 3), "cores": O.threads(),
                                          "sample": "clips 0, 97 and 201 (%d samples), steady clock around the C loops"
                                                    % c_n}}
        del xs, ss, b, ys, graph

    if want("chain_short_large"):
        log("chain_short_large (C1-L)")
        w = workloads.chain_mid_short_fir()
        x = torch.from_numpy(w.x).to(dev)
        st = [(k, torch.from_numpy(c).to(dev)) for k, c in w.stages]
        s = timed(torch, lambda: tfx.chain(x, st), 20, stream)
        y = tfx.chain(x, st)[:2].cpu().numpy()
        out["chain_short_large"] = {"workload": "8 x 5,760,000, chain_short's filters (101-tap FIR | Butterworth HP, "
                                                "2 SOS), one tfx_chain call",
                                    "Msamples_per_s": round(x.numel() / s / 1e6, 1), "ms": round(s * 1e3, 4),
                                    "hbm_frac": round(8.0 * x.numel() / s / 1e9 / HBM_PEAK_GBS, 4),
                                    "rel_err_2ch": rel_err(y, O.chain(w.x[:2], w.stages)), "tolerance": 1e-4}
        del x, st

    if want("learnable"):
        log("learnable: forward, forward + backward")
        x_np, params, target = workloads.learnable()
        x = torch.from_numpy(x_np).to(dev)
        st = [(k, torch.from_numpy(c).to(dev)) for k, c in target]
        gup = torch.from_numpy(np.random.default_rng(12).standard_normal(x_np.shape).astype(np.float32)).to(dev)
        s_f = timed(torch, lambda: tfx.chain(x, st), 20, stream)

        def fb():
            yv, ck = tfx.chain(x, st, return_ckpt=True)
            return tfx.chain_backward(x, gup, st, ck)
        s_fb = timed(torch, fb, 20, stream)
        out["learnable_fwd_bwd"] = {"workload": "64 x 192,000 (32 x 2 ch), 255-tap FIR | 8 SOS",
                                    "fwd_Msamples_per_s": round(x.numel() / s_f / 1e6, 1), "fwd_ms": round(s_f * 1e3, 4),
                                    "fwd_bwd_Msamples_per_s": round(x.numel() / s_fb / 1e6, 1),
                                    "fwd_bwd_ms": round(s_fb * 1e3, 4), "ratio_to_fwd": round(s_f / s_fb, 4),
                                    "step": "tfx_chain (+ checkpoints) and tfx_chain_backward for a fixed upstream "
                                            "gradient (input, taps and section gradients)"}
        del x, st, gup

    if want("learnable"):
        log("learnable fwd+bwd")
        x_np, params, target = workloads.learnable()
        x = torch.from_numpy(x_np).to(dev)
        hh = torch.from_numpy(params["h"]).to(dev).requires_grad_(True)
        sec = torch.from_numpy(target[1][1]).to(dev).requires_grad_(True)
        tgt = torch.from_numpy(O.chain(x_np, target).astype(np.float32)).to(dev)

        def step():
            yv = tfx.chain(x, [("fir", hh), ("sos", sec)])
            loss = torch.mean((yv - tgt) ** 2)
            loss.backward()
        s = timed(torch, step, 10, stream)
        out["learnable"] = {"workload": "64 x 192,000, 255-tap FIR + 8 SOS, MSE loss, grads of taps and sections",
                            "fwd_bwd_ms": round(s * 1e3, 3), "Msamples_per_s": round(x.numel() / s / 1e6, 1)}
        del x, hh, sec, tgt

    if want("wave_pipe"):
        log("wave pipe")
        w = workloads.chain_mid()
        x = torch.from_numpy(w.x).to(dev)
        fs = [tfx.WindowedSincFIR(300.0, num_taps=1023, cutoff_hi=6000.0), tfx.HiShelving(1000.0), tfx.LoShelving(2000.0),
              tfx.Peaking(3000.0, q=2.0, gain_db=-3.0)]

        def piped():
            wv = tfx.Wave(x, 48000.0)
            for f in fs:
                wv = wv | f
            return wv.y
        yp = piped()
        st = [f.stage(x.device) for f in fs]
        s_p = timed(torch, piped, 10, stream)
        s_c = timed(torch, lambda: tfx.chain(x, st), 10, stream)
        ref = O.chain(w.x[:2], [(f.kind, f.coefficients("cpu").numpy()) for f in fs])
        out["wave_pipe"] = {"workload": "8 x 5,760,000 @48 kHz: Wave | WindowedSincFIR(1023) | HiShelving | LoShelving "
                                        "| Peaking (one fused launch)",
                            "Msamples_per_s": round(x.numel() / s_p / 1e6, 1), "ms": round(s_p * 1e3, 4),
                            "direct_chain_ms": round(s_c * 1e3, 4),
                            "rel_err_2ch": rel_err(yp[:2].cpu().numpy(), ref), "tolerance": 1e-4}
        del x, yp

    if want("chain_mid_compute"):
        log("chain_mid, matrix-core FIR")
        w = workloads.chain_mid()
        x = torch.from_numpy(w.x).to(dev)
        st = [(k, torch.from_numpy(c).to(dev)) for k, c in w.stages]
        ref = O.chain(w.x[:2], w.stages)
        res = {"workload": "chain_mid (8 x 5,760,000, 1023-tap FIR | 6 SOS), one tfx_chain call (prepare + run)"}
        for comp in ("f32", "bf16", "f16"):
            s_c = timed(torch, lambda: tfx.chain(x, st, compute=comp), 10, stream)
            yc = tfx.chain(x, st, compute=comp)[:2].cpu().numpy()
            res[comp] = {"ms": round(s_c * 1e3, 4), "Msamples_per_s": round(x.numel() / s_c / 1e6, 1),
                         "rel_err_2ch": rel_err(yc, ref), "tolerance": 1e-4 if comp == "f32" else 1e-2}
        out["chain_mid_compute"] = res
        del x, st

    if want("stream"):
        log("stream")
        w = workloads.chain_mid(C=8, N=48000)
        x = torch.from_numpy(w.x).to(dev)
        st = [(k, torch.from_numpy(c).to(dev)) for k, c in w.stages]
        res = {"workload": "8 ch @48 kHz, chain_mid's filters (1023-tap FIR | 6 SOS), blocks carried by tfx_chain_stream"}
        for blk in (512, 4096):
            sm = tfx.ChainStream(st, 8, blk)
            nb = x.shape[1] // blk
            blocks = [x[:, i * blk:(i + 1) * blk].contiguous() for i in range(nb)]
            ys = [sm.process(b) for b in blocks]
            y = torch.cat(ys, dim=1).cpu().numpy()
            sm.reset()
            it = iter(range(10 ** 9))

            def one():
                i = next(it) % nb
                if i == 0:
                    sm.reset()
                sm.process(blocks[i])
            s = timed(torch, one, 200, stream)
            res["block_%d" % blk] = {"us_per_block": round(s * 1e6, 1), "Msamples_per_s": round(8 * blk / s / 1e6, 1),
                                     "realtime_factor": round(blk / 48000.0 / s, 1),
                                     "rel_err_vs_oracle": rel_err(y, O.chain(w.x[:, :nb * blk], w.stages)),
                                     "tolerance": 1e-4}
        out["stream"] = res
        del x

    if want("stft"):
        out["stft"] = stft_leg(torch, dev, stream)
    return out


def stft_leg(torch, dev, stream):
    """STFT and inverse STFT of the headline signal (n_fft 2048, hop 512,
    periodic Hann, centred), timed through the C ABI on resident buffers."""
    from paper_2504_08624_amd import workloads
    log("stft")
    from oracle import stft as OS
    from paper_2504_08624_amd import lib, spectral
    w = workloads.chain_mid()
    x = torch.from_numpy(w.x).to(dev)
    C, N = x.shape
    n_fft, hop = 2048, 512
    T = spectral.num_frames(N, n_fft, hop, True)
    F = n_fft // 2 + 1
    win_np = OS.hann(n_fft).astype(np.float32)
    win = torch.from_numpy(win_np).to(dev)
    spec = torch.empty((C, T, F), dtype=torch.complex64, device=dev)
    yi = torch.empty_like(x)
    sp = stream.cuda_stream

    def fwd():
        lib.call("tfx_stft", x.data_ptr(), C, N, N, n_fft, hop, win.data_ptr(), n_fft, 1, 0, spec.data_ptr(), sp)

    def inv():
        lib.call("tfx_istft", spec.data_ptr(), C, T, n_fft, hop, win.data_ptr(), n_fft, 1, 0, yi.data_ptr(), N, N, sp)
    s_f = timed(torch, fwd, 20, stream)
    s_i = timed(torch, inv, 20, stream)
    fwd()
    inv()
    g = np.random.default_rng(9)
    picks = [(int(g.integers(C)), int(g.integers(T))) for _ in range(16)] + [(0, 0), (C - 1, T - 1)]
    got = np.stack([spec[c, t].cpu().numpy() for c, t in picks])
    ref = np.stack([OS.frame(w.x[c], n_fft, hop, win_np, True, t) for c, t in picks])
    e_f = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    e_i = rel_err(yi[:, :200000].cpu().numpy(), w.x[:, :200000])
    b_f = C * N * 4 + C * T * F * 8
    b_i = C * T * F * 8 + C * N * 4
    return {"workload": "8 x 5,760,000 (chain_mid's signal), n_fft 2048, hop 512, periodic Hann, centred",
            "frames": T,
            "stft": {"ms": round(s_f * 1e3, 4), "Msamples_per_s": round(C * N / s_f / 1e6, 1),
                     "alg_GBps": round(b_f / s_f / 1e9, 1), "hbm_frac": round(b_f / s_f / 1e9 / HBM_PEAK_GBS, 4),
                     "rel_err_18_frames": e_f, "tolerance": 1e-5},
            "istft": {"ms": round(s_i * 1e3, 4), "Msamples_per_s": round(C * N / s_i / 1e6, 1),
                      "alg_GBps": round(b_i / s_i / 1e9, 1), "hbm_frac": round(b_i / s_i / 1e9 / HBM_PEAK_GBS, 4),
                      "round_trip_rel_err": e_i, "tolerance": 1e-5}}


def main():
    args = parse()
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU only (--gpus %d requested); "
              "the channels of a multi-GPU job would shard with no communication." % args.gpus,
              file=sys.stderr)
        sys.exit(2)

    import torch

    import paper_2504_08624_amd as tfx
    from paper_2504_08624_amd import lib, workloads
    from paper_2504_08624_amd.functional import _stages

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    if args.stft_only:
        print(json.dumps({"stft": stft_leg(torch, dev, torch.cuda.current_stream(dev))}))
        return
    if args.leg:
        print(json.dumps(secondary(torch, dev, torch.cuda.current_stream(dev), set(args.leg))))
        return
    log("generating chain_mid inputs (8 x 5,760,000)")
    w = workloads.chain_mid()
    C, N = w.x.shape
    x = torch.from_numpy(w.x).to(dev)
    y = torch.empty_like(x)
    kept, desc = _stages(w.stages, dev)
    arr = lib.stage_array(desc)
    nst = len(desc)
    L = lib.load()
    nb = lib.size_out()
    lib.call("tfx_chain_workspace_size", C, N, arr, nst, 0, nb)
    ws = torch.empty(max(nb.value, 256), dtype=torch.uint8, device=dev)
    stream = torch.cuda.current_stream(dev)
    sp = stream.cuda_stream

    def prepare():
        lib.check(L.tfx_chain_prepare(C, N, arr, nst, 0, ws.data_ptr(), ws.numel(), sp), "tfx_chain_prepare")

    def run():
        lib.check(L.tfx_chain_run(x.data_ptr(), y.data_ptr(), C, N, N, N, arr, nst, 0, None,
                                  ws.data_ptr(), ws.numel(), sp), "tfx_chain_run")

    # device status word of the workspace, folded after every run (before the
    # next prepare clears it): a look-back that gave up would flag it
    flags = torch.zeros(1, dtype=torch.int32, device=dev)

    def fold():
        lib.check(L.tfx_workspace_status(ws.data_ptr(), ws.numel(), flags.data_ptr(), 1, sp), "tfx_workspace_status")

    log("warmup %d" % args.warmup)
    for _ in range(args.warmup):
        prepare()
        run()
    torch.cuda.synchronize()

    K = args.steps
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(K)]
    ev0 = [torch.cuda.Event(enable_timing=True) for _ in range(K)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(K):
        ev0[i].record(stream)
        prepare()
        ev[i][0].record(stream)
        run()
        ev[i][1].record(stream)
        fold()
    torch.cuda.synchronize()
    if int(flags.item()) != 0:
        raise RuntimeError("a timed step flagged its workspace (status word 0x%x)" % int(flags.item()))
    t1 = time.perf_counter()
    wall = t1 - t0
    kern_ms = np.array([a.elapsed_time(b) for a, b in ev])
    step_ms = np.array([a.elapsed_time(b[1]) for a, b in zip(ev0, ev)])
    log("timed %d forward steps in %.3f s" % (K, wall))

    # cold steps: 512 MB written between steps so no input is left in the
    # 256 MB last-level cache (the headline input is 184 MB)
    flush = torch.empty(128 * 1024 * 1024, dtype=torch.float32, device=dev)
    cold = []
    for i in range(10):
        flush.fill_(float(i))
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(stream)
        prepare()
        run()
        b.record(stream)
        fold()
        torch.cuda.synchronize()
        cold.append(a.elapsed_time(b))
    del flush
    log("timed 10 cold steps")

    samples = C * N
    ms_step = wall / K * 1e3
    value = samples / (wall / K) / 1e6
    alg_bytes = 8.0 * samples
    memory = max(int(ws[:32].view(torch.int32)[4]) - 1, 0)   # header word: memory | 1, 0 for a scan
    fps = chain_flops_per_sample(C, N, memory)
    kern_s = float(kern_ms.mean()) / 1e3
    achieved_gbs = alg_bytes / kern_s / 1e9
    achieved_tfs = fps * samples / kern_s / 1e12 if fps else None
    out = y.cpu().numpy()

    # achievable copy bandwidth: a plain device copy of the input (also the
    # calibration of the HBM counters)
    z = torch.empty_like(x)
    for _ in range(3):
        z.copy_(x)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record(stream)
    for _ in range(10):
        z.copy_(x)
    b.record(stream)
    torch.cuda.synchronize()
    cs = a.elapsed_time(b) / 10 / 1e3
    copy = {"bytes": 2 * 4 * samples, "us": round(cs * 1e6, 2), "GBps": round(2 * 4 * samples / cs / 1e9, 1)}
    del z

    # forward + backward on the same workload
    st = [(k, t) for (k, _), t in zip(w.stages, kept)]
    g = torch.from_numpy(np.random.default_rng(11).standard_normal((C, N)).astype(np.float32)).to(dev)

    def fwd_bwd():
        yv, ck = tfx.chain(x, st, return_ckpt=True)
        return tfx.chain_backward(x, g, st, ck)
    for _ in range(args.warmup):
        fwd_bwd()
    torch.cuda.synchronize()
    kb = max(5, K // 5)
    t0 = time.perf_counter()
    for _ in range(kb):
        fwd_bwd()
    torch.cuda.synchronize()
    fb = (time.perf_counter() - t0) / kb
    log("timed %d forward+backward steps" % kb)
    fwd_bwd_rec = {"Msamples_per_s": round(samples / fb / 1e6, 3), "ms_per_step": round(fb * 1e3, 4),
                   "ratio_to_fwd": round((samples / fb / 1e6) / value, 4),
                   "step": "tfx_chain with checkpoints + tfx_chain_backward (input, taps, sections)"}
    del g

    sec = None
    if not args.quick:
        sec = secondary(torch, dev, stream)

    cpu = None
    err = None
    if not args.no_cpu_baseline:
        from oracle import oracle as O
        O.build()
        threads = min(C, O.threads())
        Ns = N  # the whole input: a few seconds of CPU work
        log("oracle on 8 x %d samples (%d threads)" % (Ns, threads))

        def oracle_chain(xs):
            """The oracle's chain, stage by stage; returns (y, seconds of the
            C filtering loops, steady clock)."""
            yv, sec = xs, 0.0
            for kind, coef in w.stages:
                yv = O.chain(yv, [(kind, coef)])
                sec += O.last_seconds()
            return yv, sec
        ref, c_sec = oracle_chain(w.x[:, :Ns])
        cpu = {"value": round(C * Ns / c_sec / 1e6, 3), "unit": "Msamples/s", "cores": threads,
               "kind": "oracle", "cpu_model": cpu_model(),
               "sample": "the whole headline input (8 x 5,760,000), whole chain, FP64, one thread per channel; "
                         "steady clock around the C loops, %.2f s" % c_sec}
        err = rel_err(out[:, :Ns], ref)
        _, c_sec1 = oracle_chain(w.x[:1, :Ns])  # one channel: one thread
        cpu["single_thread"] = {"value": round(Ns / c_sec1 / 1e6, 3), "unit": "Msamples/s",
                                "sample": "channel 0 (5,760,000 samples), whole chain, FP64, %.2f s" % c_sec1}

    rec = {
        "metric": "Msamples/s (ch x samples) fwd and fwd+bwd, % HBM roofline, at stated error",
        "value": round(value, 3),
        "unit": "Msamples/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": args.warmup,
        "ms_per_step": round(ms_step, 4),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": "chain_mid: 8 ch x 5,760,000 samples @48 kHz, 1/f noise + log sweep; "
                               "FIR 1023-tap band-pass | Chebyshev-I 8th order (4 SOS) | 2 peaking EQ",
                   "channels": C, "samples": N, "fir_taps": int(w.stages[0][1].size),
                   "sections": int(sum(s[1].shape[0] for s in w.stages if s[0] == "sos")),
                   "fir_algo": "fft", "step": "tfx_chain_prepare + tfx_chain_run"},
        "roofline": {"bound": "hbm", "achieved": round(achieved_gbs, 2), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(achieved_gbs / HBM_PEAK_GBS, 4), "traffic": measured_traffic(),
                     "kernel": "short16k_kernel (FIR and cascade as one FIR on 16384-point blocks)",
                     "kernel_us": round(kern_s * 1e6, 2),
                     "alg_bytes_per_launch": alg_bytes, "alg_bytes_per_sample": 8,
                     "copy_GBps": copy["GBps"], "frac_of_copy": round(achieved_gbs / copy["GBps"], 4),
                     "valu": {"what": "the block kernel's algorithmic flops (two 16384-point transforms and a "
                                      "spectrum product per two tiles) on the vector units, without packed fp32",
                              "memory": memory, "flops_per_sample": round(fps, 2),
                              "achieved_TFLOP_per_s": round(achieved_tfs, 3), "peak_TFLOP_per_s": VALU_F32_PEAK_TFS,
                              "frac": round(achieved_tfs / VALU_F32_PEAK_TFS, 4)} if fps else None},
        "step_stats_ms": {"median": round(float(np.median(step_ms)), 4), "mean": round(float(step_ms.mean()), 4),
                          "sd": round(float(step_ms.std(ddof=1)) if K > 1 else 0.0, 4),
                          "cold_median": round(float(np.median(cold)), 4),
                          "timing": "HIP events per step on the launch stream; cold = 512 MB written before each"},
        "fwd_bwd": fwd_bwd_rec,
        "cpu_baseline": cpu,
        "max_rel_err_vs_oracle": err,
        "tolerance": 1e-4,
    }
    if sec is not None:
        rec["secondary"] = sec
    rec["copy"] = copy
    print(json.dumps(rec), flush=True)


if __name__ == "__main__":
    main()
