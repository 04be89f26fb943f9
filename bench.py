"""Benchmark: FFT beamforming of the CHIME-shaped workload on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--skip-extras] [--skip-cpu]

One step = one bf_beamform_fft call over the whole workload: 4 x 256 lattice,
2 polarisations, 256 channels, 16384 samples of int4+4 voltages (8 GiB,
resident in HBM before timing), E-W 4-point DFT, N-S transform zero-padded to
512, |B|^2 summed over 16 samples, 256 N-S beams kept per channel (2 GiB of
FP32 intensities).  Prints one JSON line.
"""
from __future__ import annotations

import argparse
import contextlib
import gc
import hashlib
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "beamformed antenna-samples/s FP32 FFT vs FP16/FP8-MFMA; %HBM peak; tied-beam p99 ms"
HBM_PEAK_GBS = 8000.0
FP32_VECTOR_PEAK_TFLOPS = 157.3
BF16_MFMA_PEAK_TFLOPS = 2500.0
INT8_MFMA_PEAK_TOPS = 5000.0
N_SIMD = 256 * 4       # 256 compute units x 4 SIMDs
CLOCK_HZ = 2.4e9        # peak engine clock


def flops_per_frame(n_ns: int, m_ns: int, keep: int, m_ew: int = 4) -> float:
    """Nominal algorithmic flops for one (sample, channel, polarisation) frame.

    N-S transform counted as 5 M log2 M per E-W beam (the usual FFT
    convention), the E-W 4-point DFT as its 16 real additions per N-S
    position, |B|^2 plus accumulation as 4 flops per kept beam.
    """
    return m_ew * 5 * m_ns * math.log2(m_ns) + 16 * n_ns + 4 * m_ew * keep


def lag_products(frames: int) -> float:
    """int8 operations that the stacked visibilities of a 4 x 256 lattice issue: per 16 samples and E-W beam 160 of
    v_mfma_i32_16x16x64_i8 (the upper half of the 256 x 256 products in 16 x 16 tiles, real and imaginary parts)."""
    return frames / 16 * 4 * 160 * (16 * 16 * 64 * 2)


def kernel_source_hash(*names) -> str:
    """Hash of the kernel sources with comments and whitespace removed, so a
    profile stays matched to the code it measured across comment edits."""
    import re
    h = hashlib.sha256()
    for n in names:
        with open(os.path.join(ROOT, "paper_1710_08591_amd", "csrc", n), encoding="utf-8") as f:
            src = f.read()
        src = re.sub(r"/\*.*?\*/", " ", src, flags=re.S)
        src = re.sub(r"//[^\n]*", " ", src)
        h.update(" ".join(src.split()).encode())
    return h.hexdigest()[:16]


def counters_from_profile(name: str, src_hash: str) -> dict:
    """Counter readings per launch stored under profiles/, if they were taken
    on the current kernel source (else an empty dict)."""
    p = os.path.join(ROOT, "profiles", name)
    if not os.path.exists(p):
        return {}
    try:
        d = json.load(open(p))
    except Exception:
        return {}
    if d.get("kernel_source_hash") != src_hash:
        return {}
    return d


class OracleChecks:
    """Sampled GPU outputs awaiting comparison with the FP64 oracle.

    The measurement legs only record what they computed: host copies of a
    few output slices and the inputs that define them.  Every oracle call
    happens in the oracle leg (``cpu_baseline``), which writes the largest
    error of each group back into the measurement's record (``None`` when
    the oracle leg is skipped)."""

    def __init__(self):
        self.items = []

    def add(self, rec: dict, key: str, kind: str, got, n_slices: int = 1, **args):
        import numpy as np
        rec.setdefault(key, None)
        self.items.append((rec, key, kind, np.asarray(got, dtype=np.float64), dict(args, n_slices=n_slices)))

    def add_blocks(self, rec: dict, key: str, out, w, blocks=None, **ref_args):
        """Whole blocks of a CHIME-shaped output (every channel and both
        polarisations, each channel's own clamp table), the first and the last
        by default."""
        blocks = (0, w.n_time // w.block - 1) if blocks is None else blocks
        for blk in blocks:
            self.add(rec, key, "fft_rel", out[blk].cpu().numpy(), n_slices=w.n_chan * w.n_pol,
                     v=host_block(w, blk), m_ew=w.m_ew, m_ns=w.m_ns, ns_select=w.ns_select(), index=(0,),
                     **ref_args)


_HOST_BLOCKS = {}


def host_block(w, blk: int):
    """One whole block of the workload's voltages (every channel and
    polarisation) on the host, from the seeded generator; kept for reuse."""
    import synthgen as sg
    key = (repr(w), blk)
    if key not in _HOST_BLOCKS:
        _HOST_BLOCKS[key] = sg.volts(w, blk * w.block, w.block)
    return _HOST_BLOCKS[key]


def _host_statement() -> dict:
    """What the oracle ran on: CPU model, logical CPUs, the CPUs this process
    may use, the thread variables of the environment and the BLAS pools."""
    model = None
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    try:
        affinity = len(os.sched_getaffinity(0))
    except Exception:
        affinity = None
    env = {k: os.environ.get(k) for k in ("OMP_NUM_THREADS", "OPENBLAS_NUM_THREADS", "MKL_NUM_THREADS",
                                          "BLIS_NUM_THREADS", "NUMEXPR_NUM_THREADS")}
    try:
        from threadpoolctl import threadpool_info
        pools = [{"api": i.get("internal_api"), "threads": i.get("num_threads"), "version": i.get("version")}
                 for i in threadpool_info()]
    except Exception:
        pools = []
    return {"cpu_model": model, "nproc": os.cpu_count(), "cpus_allowed": affinity, "thread_env": env,
            "blas_pools": pools}


def cpu_baseline(seconds: float = 15.0, checks: "OracleChecks | None" = None, seconds_1t: float = 8.0):
    """The FP64 oracle: timed on a bounded slice of the same workload on the
    host cores (all BLAS threads, then one thread on the first of the same
    slices), then compared with every sampled GPU output in ``checks``."""
    import numpy as np

    import oracle as orc
    import synthgen as sg
    host = _host_statement()
    cores = max([p["threads"] or 1 for p in host["blas_pools"]] or [1])
    w = sg.make_workload("c2")
    sel = w.ns_select()
    chunk = 1024
    slices = []

    def one(k):
        c = (37 * k) % w.n_chan
        p = k % w.n_pol
        t_lo = (k * chunk) % w.n_time
        if k == len(slices):
            slices.append(sg.volts(w, t_lo, chunk, chans=[c], pols=[p]))
        ts = time.perf_counter()
        i = orc.beamform_fft(slices[k], w.m_ew, w.m_ns, w.block)[..., sel[c]]
        dt = time.perf_counter() - ts
        assert i.shape == (chunk // 16, 1, 1, 4, 256)
        return dt

    n_cp = 0
    elapsed = 0.0
    while elapsed < seconds:
        elapsed += one(n_cp)
        n_cp += 1
    done = n_cp * chunk * w.n_ant
    # one thread, on the first slices of the same list
    n_1t = 0
    el_1t = 0.0
    try:
        from threadpoolctl import threadpool_limits
        with threadpool_limits(limits=1):
            while el_1t < seconds_1t and n_1t < n_cp:
                el_1t += one(n_1t)
                n_1t += 1
        rate_1t = n_1t * chunk * w.n_ant / el_1t
    except Exception:
        rate_1t = None
    slices.clear()
    rec = {"value": done / elapsed, "unit": "antenna-samples/s", "cores": int(cores), "kind": "oracle",
           "sample": f"{n_cp} slices of {chunk} samples x 1 channel x 1 pol of the 4x256 lattice "
                     f"({done} antenna-samples, {elapsed:.1f} s of oracle time, generation excluded)",
           "value_1_thread": rate_1t,
           "sample_1_thread": f"the first {n_1t} of the same slices with the BLAS pools limited to one thread "
                              f"({el_1t:.1f} s)",
           **host}

    def reference(kind, a):
        if kind == "fft_rel":
            r = orc.beamform_fft(a["v"], a["m_ew"], a["m_ns"], 16, taper=a.get("taper"),
                                 ns_select=a.get("ns_select"))[a.get("index", ())]
            return r if a.get("sel") is None else r[..., a["sel"]]
        if kind == "tied_rel":
            r = orc.tied_intensity(a["v"], a["dircos"], a["dl"], 16, chans=[a["c"]])[0, 0]
            return r if a.get("shape") is None else r.reshape(a["shape"])
        if kind == "regrid_prop":
            b = orc.beamform_fft(a["v"], a["m_ew"], a["m_ns"], 16)[0, 0]
            if a["weights"] == "paper":
                W = np.stack([orc.regrid_weights_paper(a["n_ns"], a["m_ns"], y) for y in a["ys"]])
            else:
                full = orc.optimal_window_weights(a["h"], a["m_ns"], a["ys"])
                W = np.zeros_like(full)
                for t, y in enumerate(a["ys"]):
                    if a["k"]:
                        first, taps = orc.compact_taps(full[t], y, a["k"])
                        W[t, (first + np.arange(a["k"])) % a["m_ns"]] = taps
                    else:
                        W[t] = full[t]
            return orc.regrid_intensity(b, W), orc.regrid_intensity(b, np.abs(W))
        if kind == "localize_abs":
            x = orc.beamform_fft(a["v"], a["m_ew"], a["m_ns"], 16)
            st, _ = orc.localize(x, a["n_ns"], a["dl_ns"], a["n_window"], a["n_iter"], chans=[a["c"]])
            return st
        raise ValueError(kind)

    n_checked = 0
    for target, key, kind, got, a in (checks.items if checks else []):
        ref = reference(kind, a)
        if kind == "regrid_prop":
            err = float(np.max(np.abs(got - ref[0]) / ref[1]))
        elif kind == "localize_abs":
            err = float(np.max(np.abs(got - ref)))
        else:
            err = float(np.max(np.abs(got - ref) / ref))
        target[key] = err if target.get(key) is None else max(target[key], err)
        n_checked += a["n_slices"]
    rec["parity_slices_checked"] = n_checked
    return rec


def _leg(fn, *args):
    """Run one side measurement; an exception in it is reported in its record
    instead of taking the headline line down with it."""
    try:
        return fn(*args)
    except Exception as e:
        import traceback
        traceback.print_exc(file=sys.stderr)
        return {"error": f"{type(e).__name__}: {e}"}


@contextlib.contextmanager
def _no_gc():
    """Python's cyclic garbage collector held off inside a timed region: a
    collection pauses the host, and once the launch queue has drained the
    GPU idles between the events that bracket the launches."""
    gc.collect()
    gc.disable()
    try:
        yield
    finally:
        gc.enable()


def _time_launches(fn, n: int, warmup: int = 2, each: list = None, warm_ms: float = 500.0) -> float:
    """Average milliseconds of fn() (one launch on the current stream);
    with ``each`` the time of every launch is appended to it.  Warm-up runs
    at least ``warmup`` launches and at least ``warm_ms`` of them (up to 400
    launches), so that the clocks have left an idle state before the timed
    launches (the host-side checks between legs leave the GPU idle), and the
    first timed launch is queued behind two more, not after a synchronisation
    (after one, a 14 ms launch read 17 ms)."""
    import torch
    t0 = time.perf_counter()
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    done = warmup
    while (time.perf_counter() - t0) * 1e3 < warm_ms and done < 400:
        fn()
        done += 1
        if done % 8 == 0:
            torch.cuda.synchronize()
    s = torch.cuda.current_stream()
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(n + 1)]
    with _no_gc():
        # two more launches queued ahead of the first event, so that the GPU
        # does not idle (and lower its clock) between warm-up and timing
        fn()
        fn()
        ev[0].record(s)
        for i in range(n):
            fn()
            ev[i + 1].record(s)
        torch.cuda.synchronize()
    if each is not None:
        each.extend(round(ev[i].elapsed_time(ev[i + 1]), 4) for i in range(n))
    return ev[0].elapsed_time(ev[n]) / n


def run_chime_mixed(dev, w, volts, fp32_ms: float, checks: OracleChecks) -> dict:
    """The same resident CHIME-shaped voltages through the FP16 and FP8 plans
    (unwindowed intensities of every precision are the same exact integer sums)
    and with a window or gains."""
    import numpy as np
    import torch

    import paper_1710_08591_amd as bf
    import synthgen as sg
    plan = bf.Plan(n_ew=w.n_ew, n_ns=w.n_ns, m_ew=w.m_ew, m_ns=w.m_ns, n_pol=w.n_pol, n_chan=w.n_chan,
                   block=w.block, ns_select=w.ns_select(), d_over_lambda=w.d_over_lambda(),
                   precision=bf.BF_PREC_FP16_MFMA)
    out = torch.empty(plan.out_shape(w.n_time), dtype=torch.float32, device=dev)
    ms = _time_launches(lambda: bf.beamform_fft(plan, volts, out=out), 10)
    rng = np.random.default_rng(3)
    sel = w.ns_select()
    rec = {}
    checks.add_blocks(rec, "max_rel_power_err_sampled", out, w)
    for _ in range(4):
        blk, c, p = int(rng.integers(1024)), int(rng.integers(256)), int(rng.integers(2))
        checks.add(rec, "max_rel_power_err_sampled", "fft_rel", out[blk, c, p].cpu().numpy(),
                   v=sg.volts(w, blk * 16, 16, chans=[c], pols=[p]), m_ew=w.m_ew, m_ns=w.m_ns,
                   index=(0, 0, 0), sel=sel[c])
    alg = w.n_time * w.n_chan * w.n_pol * w.frame_bytes + out.numel() * 4
    # the FP8 plan on the same voltages
    plan8 = bf.Plan(n_ew=w.n_ew, n_ns=w.n_ns, m_ew=w.m_ew, m_ns=w.m_ns, n_pol=w.n_pol, n_chan=w.n_chan,
                    block=w.block, ns_select=w.ns_select(), d_over_lambda=w.d_over_lambda(),
                    precision=bf.BF_PREC_FP8_MFMA)
    ms8 = _time_launches(lambda: bf.beamform_fft(plan8, volts, out=out), 5)
    plan8.close()
    fp8_rec = {"precision": "stacked visibilities as exact int8 products, FP64 transforms per block",
               "kernel_ms": ms8, "antenna_samples_per_s": w.antenna_samples / (ms8 / 1e3),
               "speedup_vs_fp32": fp32_ms / ms8}
    checks.add_blocks(fp8_rec, "max_rel_power_err_sampled", out, w)
    # the per-antenna Gaussian window on the FP16 matrix-core plan (windowed E-W sums split into hi + lo)
    hwin = np.ascontiguousarray(sg.gaussian_taper(w.n_ew, w.n_ns), dtype=np.float32)
    hwin_dev = torch.from_numpy(hwin).to(dev)
    hm_ms = _time_launches(lambda: bf.beamform_fft(plan, volts, out=out, taper=hwin_dev), 5)
    fp16_window_rec = {"kernel_ms": hm_ms, "antenna_samples_per_s": w.antenna_samples / (hm_ms / 1e3),
                       "slowdown_vs_no_window": hm_ms / ms, "speedup_vs_fp32_with_window": None}
    checks.add_blocks(fp16_window_rec, "max_rel_power_err_sampled", out, w, blocks=(0,),
                      taper=hwin.astype(np.float64))
    # complex per-antenna gains (bf_beamform_fft_gains) on the same voltages, FP32 plan
    plan32 = bf.Plan(n_ew=w.n_ew, n_ns=w.n_ns, m_ew=w.m_ew, m_ns=w.m_ns, n_pol=w.n_pol, n_chan=w.n_chan,
                     block=w.block, ns_select=w.ns_select(), d_over_lambda=w.d_over_lambda())
    grng = np.random.default_rng(17)
    gains = np.exp(0.1 * grng.normal(size=(w.n_ns, w.n_ew)) + 0.1j * grng.normal(size=(w.n_ns, w.n_ew)))
    g_dev = torch.from_numpy(gains.astype(np.complex64)).to(dev)
    g_ms = _time_launches(lambda: bf.beamform_fft(plan32, volts, out=out, gains=g_dev), 5)
    gains_rec = {"kernel_ms": g_ms, "antenna_samples_per_s": w.antenna_samples / (g_ms / 1e3),
                 "slowdown_vs_no_gains": g_ms / fp32_ms}
    checks.add_blocks(gains_rec, "max_rel_power_err_sampled", out, w, blocks=(0,),
                      taper=gains.astype(np.complex64).astype(np.complex128))
    for _ in range(2):
        blk, c, p = int(rng.integers(1024)), int(rng.integers(256)), int(rng.integers(2))
        checks.add(gains_rec, "max_rel_power_err_sampled", "fft_rel", out[blk, c, p].cpu().numpy(),
                   v=sg.volts(w, blk * 16, 16, chans=[c], pols=[p]), m_ew=w.m_ew, m_ns=w.m_ns,
                   index=(0, 0, 0), sel=sel[c], taper=gains.astype(np.complex64).astype(np.complex128))
    # the per-antenna Gaussian window (real sculpting weights) on the same voltages, FP32 plan
    h = sg.gaussian_taper(w.n_ew, w.n_ns)
    h_dev = torch.from_numpy(np.ascontiguousarray(h, dtype=np.float32)).to(dev)
    h_ms = _time_launches(lambda: bf.beamform_fft(plan32, volts, out=out, taper=h_dev), 5)
    window_rec = {"kernel_ms": h_ms, "antenna_samples_per_s": w.antenna_samples / (h_ms / 1e3),
                  "slowdown_vs_no_window": h_ms / fp32_ms}
    fp16_window_rec["speedup_vs_fp32_with_window"] = h_ms / hm_ms
    checks.add_blocks(window_rec, "max_rel_power_err_sampled", out, w, blocks=(0,),
                      taper=np.asarray(h, dtype=np.float64))
    for _ in range(2):
        blk, c, p = int(rng.integers(1024)), int(rng.integers(256)), int(rng.integers(2))
        checks.add(window_rec, "max_rel_power_err_sampled", "fft_rel", out[blk, c, p].cpu().numpy(),
                   v=sg.volts(w, blk * 16, 16, chans=[c], pols=[p]), m_ew=w.m_ew, m_ns=w.m_ns,
                   index=(0, 0, 0), sel=sel[c], taper=np.asarray(h, dtype=np.float64))
    plan32.close()
    mfma_ops = lag_products(w.n_time * w.n_chan * w.n_pol)
    plan.close()
    rec.update({"workload": "same as the headline (4x256, 2 pol, 256 chan, 16384 samples, clamp 256)",
                "precision": "stacked visibilities as exact int8 products, FP64 transforms per block",
                "kernel_ms": ms, "antenna_samples_per_s": w.antenna_samples / (ms / 1e3),
                "speedup_vs_fp32": fp32_ms / ms,
                "hbm_alg_gbs": alg / (ms / 1e3) / 1e9, "hbm_frac": alg / (ms / 1e3) / 1e9 / HBM_PEAK_GBS,
                "mfma_int8_tops": mfma_ops / (ms / 1e3) / 1e12,
                "mfma_frac_of_int8_peak": mfma_ops / (ms / 1e3) / 1e12 / INT8_MFMA_PEAK_TOPS,
                "fp8_mfma": fp8_rec, "fp16_mfma_with_real_window": fp16_window_rec,
                "fp32_with_complex_gains": gains_rec, "fp32_with_real_window": window_rec})
    return rec


def run_chime_coadding(dev, w, volts, fp32_ms: float, checks: OracleChecks) -> dict:
    """Cyclic co-adding (fewer N-S beams than antennas): the same resident
    voltages, 256 N-S antennas summed a mod m onto m = 128 and 64 positions
    before an m-point transform, unclamped FP32 plans, sampled outputs against
    the oracle's beams over all 256 antennas."""
    import numpy as np
    import torch

    import paper_1710_08591_amd as bf
    import synthgen as sg
    rng = np.random.default_rng(29)
    frames = w.n_time * w.n_chan * w.n_pol
    rec = {"workload": "same voltages as the headline (4x256, 2 pol, 256 chan, 16384 samples), m_ns < n_ns, no clamp"}
    for m in (128, 64):
        plan = bf.Plan(n_ew=w.n_ew, n_ns=w.n_ns, m_ew=w.m_ew, m_ns=m, n_pol=w.n_pol, n_chan=w.n_chan,
                       block=w.block, d_over_lambda=w.d_over_lambda())
        out = torch.empty(plan.out_shape(w.n_time), dtype=torch.float32, device=dev)
        ms = _time_launches(lambda: bf.beamform_fft(plan, volts, out=out), 5)
        # nominal: the m-point transform per E-W beam, the E-W DFT, the
        # co-adding of n_ns onto m positions (2 flop per complex addition)
        # and |B|^2 plus accumulation per beam
        flops = frames * (w.m_ew * 5 * m * math.log2(m) + 16 * w.n_ns + 2 * w.m_ew * (w.n_ns - m)
                          + 4 * w.m_ew * m)
        alg = frames * w.frame_bytes + out.numel() * 4
        r = {"kernel_ms": ms, "antenna_samples_per_s": w.antenna_samples / (ms / 1e3),
             "vs_headline_ms": ms / fp32_ms,
             "alu_tflops_nominal": flops / (ms / 1e3) / 1e12,
             "alu_frac_nominal": flops / (ms / 1e3) / 1e12 / FP32_VECTOR_PEAK_TFLOPS,
             "hbm_alg_gbs": alg / (ms / 1e3) / 1e9, "hbm_frac": alg / (ms / 1e3) / 1e9 / HBM_PEAK_GBS}
        for _ in range(2):
            blk, c, p = int(rng.integers(w.n_time // w.block)), int(rng.integers(w.n_chan)), int(rng.integers(w.n_pol))
            checks.add(r, "max_rel_power_err_sampled", "fft_rel", out[blk, c, p].cpu().numpy(),
                       v=sg.volts(w, blk * w.block, w.block, chans=[c], pols=[p]), m_ew=w.m_ew, m_ns=m,
                       index=(0, 0, 0))
        rec[f"m_ns_{m}"] = r
        plan.close()
        del out
        torch.cuda.empty_cache()
    return rec


def run_library_fft_comparator(dev, w, volts, plan, fp32_ms: float, chunk: int = 1024) -> dict:
    """Context only, not the product: the same CHIME-shaped step written with
    torch's FFT (rocFFT) and elementwise ops on the resident voltages -- decode
    to complex64, 2-D FFT with the N-S axis zero-padded to M, |B|^2, block sum,
    clamp -- timed on a slice of the samples and scaled to the whole workload."""
    import torch
    sel = torch.from_numpy(w.ns_select()).to(dev).long()                  # [chan][keep]
    v = volts[:chunk]

    def step():
        b = v.to(torch.int16)
        re = ((b >> 4) ^ 8) - 8                                          # signed high nibble
        im = ((b & 15) ^ 8) - 8                                          # signed low nibble
        x = torch.complex(re.float(), im.float())                        # [T][chan][pol][ns][ew]
        f = torch.fft.fft2(x, s=(w.m_ns, w.m_ew), dim=(-2, -1))          # [T][chan][pol][M][4]
        i = (f.real ** 2 + f.imag ** 2).view(chunk // w.block, w.block, *f.shape[1:]).sum(1)
        i = i.transpose(-1, -2)                                          # [blk][chan][pol][4][M]
        idx = sel.view(1, w.n_chan, 1, 1, w.keep).expand(i.shape[0], w.n_chan, w.n_pol, w.m_ew, w.keep)
        return torch.gather(i, -1, idx) / float(w.n_ew * w.n_ns)

    ms = _time_launches(step, 3, warmup=1)
    full_ms = ms * (w.n_time / chunk)
    import paper_1710_08591_amd as bf
    ours = bf.beamform_fft(plan, v)
    theirs = step()
    agree = float(((ours.double() - theirs.double()).abs() / theirs.double()).max())
    return {"what": "context only: torch.fft (rocFFT) and torch elementwise ops, not the product",
            "slice": f"{chunk} of {w.n_time} samples, all channels and pols; time scaled by {w.n_time // chunk}",
            "ms_per_slice": ms, "ms_scaled_to_workload": full_ms,
            "antenna_samples_per_s": w.antenna_samples / (full_ms / 1e3),
            "fused_kernel_speedup": full_ms / fp32_ms,
            "max_rel_diff_vs_fused_kernel_on_slice": agree}


def run_chime_regrid(dev, w, volts, fp32_ms: float, checks: OracleChecks, n_target: int = 256) -> dict:
    """All 512 N-S FFT beams of the resident CHIME-shaped voltages (no clamp),
    regridded to n_target achromatic N-S steering angles (eq. e:bp_max_arbitrary)."""
    import numpy as np
    import torch

    import paper_1710_08591_amd as bf
    import synthgen as sg
    plan = bf.Plan(n_ew=w.n_ew, n_ns=w.n_ns, m_ew=w.m_ew, m_ns=w.m_ns, n_pol=w.n_pol, n_chan=w.n_chan,
                   block=w.block, d_over_lambda=w.d_over_lambda())
    st = np.linspace(-0.95, 0.95, n_target)
    rg = bf.Regrid(plan, st)
    fft_i = torch.empty(plan.out_shape(w.n_time), dtype=torch.float32, device=dev)
    fft_ms = _time_launches(lambda: bf.beamform_fft(plan, volts, out=fft_i), 5)
    n_blk = w.n_time // w.block
    out = torch.empty((n_blk, w.n_chan, w.n_pol, w.m_ew, n_target), dtype=torch.float32, device=dev)
    ms = _time_launches(lambda: rg(fft_i, out=out), 10)
    rng = np.random.default_rng(5)
    dl = w.d_over_lambda()
    rec = {}
    for _ in range(3):
        blk, c = int(rng.integers(n_blk)), int(rng.integers(w.n_chan))
        vs = sg.volts(w, blk * 16, 16, chans=[c])
        e = np.repeat(np.arange(w.m_ew), n_target)
        dircos = np.stack([e / (w.m_ew * dl[c, 0]), np.tile(st, w.m_ew)], axis=1)
        got = out[blk, c].cpu().numpy()
        checks.add(rec, "max_rel_power_err_sampled", "tied_rel", got, v=vs, dircos=dircos, dl=dl, c=c,
                   shape=(w.n_pol, w.m_ew, n_target))
        checks.add(rec, "max_err_over_sum_abs_w_b_sampled", "regrid_prop", got, v=vs, m_ew=w.m_ew, m_ns=w.m_ns,
                   weights="paper", n_ns=w.n_ns, ys=dl[c, 1] * st)
    rows = n_blk * w.n_chan * w.n_pol * w.m_ew
    flops = 2.0 * rows * w.m_ns * n_target
    alg = 4.0 * rows * (w.m_ns + n_target) + 4.0 * w.n_chan * n_target * w.m_ns
    rg.close()
    # the optimally windowed beam (eq. e:wA_windowed), dense and with the compact 5-tap kernel
    h = np.sin(np.pi * (np.arange(w.n_ns) + 1) / (w.n_ns + 1))
    windowed = {}
    for k in (0, 5):
        rgw = bf.Regrid(plan, st, window=h, n_taps=k)
        kms = _time_launches(lambda: rgw(fft_i, out=out), 10)
        k_alg = 4.0 * rows * (w.m_ns + n_target) + (4.0 * w.n_chan * n_target * (k + 1) if k else
                                                      4.0 * w.n_chan * n_target * w.m_ns)
        wrec = windowed["dense" if k == 0 else f"compact_{k}_tap"] = {
            "kernel_ms": kms, "hbm_alg_gbs": k_alg / (kms / 1e3) / 1e9,
            "hbm_frac": k_alg / (kms / 1e3) / 1e9 / HBM_PEAK_GBS}
        for _ in range(2):
            blk, c = int(rng.integers(n_blk)), int(rng.integers(w.n_chan))
            checks.add(wrec, "max_err_over_sum_abs_w_b_sampled", "regrid_prop", out[blk, c].cpu().numpy(),
                       v=sg.volts(w, blk * 16, 16, chans=[c]), m_ew=w.m_ew, m_ns=w.m_ns, weights="window",
                       h=h, k=k, ys=dl[c, 1] * st)
        rgw.close()
    # Newton localisation of every row (Sec. "Localization"), 10-beam window, 6 updates
    st_o = torch.empty((n_blk, w.n_chan, w.n_pol, w.m_ew), dtype=torch.float64, device=dev)
    pk_o = torch.empty((n_blk, w.n_chan, w.n_pol, w.m_ew), dtype=torch.float32, device=dev)
    lib = bf.lib()
    loc_ms = _time_launches(lambda: bf.check(lib.bf_localize(plan.handle, bf._ptr(fft_i), n_blk, 10, 6,
                                                              bf._ptr(st_o), bf._ptr(pk_o),
                                                              bf._stream_handle()), "bf_localize"), 10)
    loc_bytes = 4.0 * rows * w.m_ns + 12.0 * rows
    localisation = {"workload": "every (block, channel, pol, E-W beam) row of the same unclamped intensities "
                                "(2M rows x 512 beams), 10-beam window, 6 Newton updates, FP64",
                    "kernel_ms": loc_ms, "rows_per_s": rows / (loc_ms / 1e3),
                    "hbm_alg_gbs": loc_bytes / (loc_ms / 1e3) / 1e9,
                    "hbm_frac": loc_bytes / (loc_ms / 1e3) / 1e9 / HBM_PEAK_GBS}
    for _ in range(2):
        blk, c = int(rng.integers(n_blk)), int(rng.integers(w.n_chan))
        checks.add(localisation, "max_abs_sin_theta_diff_sampled_vs_oracle_chain", "localize_abs",
                   st_o[blk:blk + 1, c:c + 1].cpu().numpy(), v=sg.volts(w, blk * 16, 16, chans=[c]),
                   m_ew=w.m_ew, m_ns=w.m_ns, n_ns=w.n_ns, dl_ns=dl[:, 1], c=c, n_window=10, n_iter=6)
    plan.close()
    # E-W axis padded to 8 beams and exact 2-D regridding to 256 pointings
    del out
    plan8 = bf.Plan(n_ew=w.n_ew, n_ns=w.n_ns, m_ew=8, m_ns=w.m_ns, n_pol=w.n_pol, n_chan=w.n_chan,
                    block=w.block, d_over_lambda=dl)
    dirs = sg.pointings(n_target, 12)
    rg2 = bf.Regrid2D(plan8, dirs)
    fft8 = torch.empty(plan8.out_shape(w.n_time), dtype=torch.float32, device=dev)
    del fft_i
    torch.cuda.empty_cache()
    fft8_ms = _time_launches(lambda: bf.beamform_fft(plan8, volts, out=fft8), 3, warmup=1)
    out2 = torch.empty((n_blk, w.n_chan, w.n_pol, n_target), dtype=torch.float32, device=dev)
    r2_ms = _time_launches(lambda: rg2(fft8, out=out2), 10)
    regrid_2d = {}
    for _ in range(2):
        blk, c = int(rng.integers(n_blk)), int(rng.integers(w.n_chan))
        checks.add(regrid_2d, "max_rel_power_err_sampled_vs_phased_beams", "tied_rel", out2[blk, c].cpu().numpy(),
                   v=sg.volts(w, blk * 16, 16, chans=[c]), dircos=dirs, dl=dl, c=c)
    # the same padded step with the per-antenna Gaussian window (one launch as well)
    hw8 = sg.gaussian_taper(w.n_ew, w.n_ns)
    hw8_dev = torch.from_numpy(np.ascontiguousarray(hw8, dtype=np.float32)).to(dev)
    fft8w_ms = _time_launches(lambda: bf.beamform_fft(plan8, volts, out=fft8, taper=hw8_dev), 3, warmup=1)
    win8 = {"kernel_ms": fft8w_ms, "vs_m_ew8_unwindowed": fft8w_ms / fft8_ms}
    for _ in range(2):
        blk, c = int(rng.integers(n_blk)), int(rng.integers(w.n_chan))
        checks.add(win8, "max_rel_power_err_sampled", "fft_rel", fft8[blk, c:c + 1].cpu().numpy(), n_slices=w.n_pol,
                   v=sg.volts(w, blk * 16, 16, chans=[c]), m_ew=8, m_ns=w.m_ns, taper=hw8.astype(np.float64),
                   index=(0,))
    rows8 = n_blk * w.n_chan * w.n_pol * 8
    flops2 = 2.0 * rows8 * w.m_ns * n_target
    regrid_2d.update({"workload": "same voltages, E-W zero-padded to 8 beams (8 x 512 FFT beams), exact 2-D "
                                  f"regridding to {n_target} pointings per channel, pol and block",
                      "fft_m_ew8_ms": fft8_ms, "fft_m_ew8_vs_headline": fft8_ms / fp32_ms,
                      "fft_m_ew8_gaussian_window": win8, "kernel_ms": r2_ms,
                      "contraction_tflops": flops2 / (r2_ms / 1e3) / 1e12,
                      "mfma_bf16_frac": 6 * flops2 / (r2_ms / 1e3) / 1e12 / BF16_MFMA_PEAK_TFLOPS})
    rg2.close()
    plan8.close()
    del fft8, out2
    rec.update({"workload": "same voltages as the headline, no clamp (512 N-S beams), regridded to "
                            f"{n_target} sin(theta) targets per E-W beam, channel and block",
                "fft_unclamped_ms": fft_ms, "kernel_ms": ms,
                "contraction_tflops": flops / (ms / 1e3) / 1e12,
                "mfma_bf16_frac": 6 * flops / (ms / 1e3) / 1e12 / BF16_MFMA_PEAK_TFLOPS,
                "hbm_alg_gbs": alg / (ms / 1e3) / 1e9, "hbm_frac": alg / (ms / 1e3) / 1e9 / HBM_PEAK_GBS,
                "optimal_window_half_sine": windowed,
                "localisation": localisation,
                "regrid_2d_m_ew8": regrid_2d})
    return rec


def run_extras(dev, checks: OracleChecks) -> dict:
    """Side-by-side precision variants, per-variant error, tied-beam throughput."""
    import numpy as np
    import torch

    import paper_1710_08591_amd as bf
    import synthgen as sg
    ex = {}
    # (1) FP32, FP16 and FP8 plans on the 4 x 16 lattice at scale
    w = sg.Workload("lattice4x16_scaled", 4, 16, 256, 2, 16384, 4, 32, 16, 6,
                    src_dircos=((0.3, -0.2), (-0.7, 0.5)), src_snr=(10.0, 30.0), dl_lo=0.4, dl_hi=0.8)
    volts = sg.volts(w, backend="torch", device=dev)
    rng = np.random.default_rng(7)
    picks = [(int(rng.integers(w.n_time // 16)), int(rng.integers(w.n_chan)), int(rng.integers(w.n_pol)))
             for _ in range(4)]
    in_b = w.n_time * w.n_chan * w.n_pol * w.frame_bytes
    variants = {}
    for prec, name in ((0, "fp32_fft"), (1, "fp16_mfma"), (2, "fp8_mfma")):
        plan = bf.Plan(n_ew=4, n_ns=16, n_pol=2, n_chan=256, block=16, precision=prec)
        out = torch.empty(plan.out_shape(w.n_time), dtype=torch.float32, device=dev)
        ms = _time_launches(lambda: bf.beamform_fft(plan, volts, out=out), 10)
        alg = in_b + out.numel() * 4
        variants[name] = {"antenna_samples_per_s": w.antenna_samples / (ms / 1e3), "kernel_ms": ms,
                          "hbm_alg_gbs": alg / (ms / 1e3) / 1e9, "hbm_frac": alg / (ms / 1e3) / 1e9 / HBM_PEAK_GBS}
        for b, c, p in picks:
            checks.add(variants[name], "max_rel_power_err_sampled", "fft_rel", out[b, c, p].cpu().numpy(),
                       v=sg.volts(w, b * 16, 16, chans=[c], pols=[p]), m_ew=4, m_ns=32, index=(0, 0, 0))
        plan.close()
        del out
    ex["precision_variants"] = {"workload": "4x16 lattice, 2 pol, 256 chan, 16384 samples (512 MiB int4+4), "
                                            "M_ns = 32, |B|^2 over 16", "variants": variants}
    del volts
    # (2) the tiny workload's bytes through each variant: error vs the FP64 oracle, every beam
    w1 = sg.make_workload("c4")
    v1 = sg.volts(w1)
    errs = {}
    for prec, name in ((0, "fp32_fft"), (1, "fp16_mfma"), (2, "fp8_mfma")):
        plan = bf.Plan(n_ew=4, n_ns=16, block=16, precision=prec)
        o = bf.beamform_fft(plan, torch.from_numpy(v1).to(dev)).cpu().numpy()
        checks.add(errs, name, "fft_rel", o, v=v1, m_ew=4, m_ns=32)
        plan.close()
    ex["tiny_workload_max_rel_power_err"] = errs
    # (3) tied-array beams from voltages: 64 pointings, 256 channels, 16384 samples, 4 x 16 lattice
    wt = sg.make_workload("c5")
    vt = sg.volts(wt, 0, 16384, backend="torch", device=dev)
    plan = bf.Plan(n_ew=4, n_ns=16, n_chan=256, block=16, d_over_lambda=wt.d_over_lambda())
    d = torch.from_numpy(sg.pointings(64, 11)).to(dev)
    ms = _time_launches(lambda: bf.form_tied_beams_v(plan, vt, 0, 256, d), 5, warmup=1)
    ex["tied_beams_v"] = {"workload": "4x16 lattice, 256 chan, 16384 samples, 64 pointings, |B|^2 over 16",
                          "kernel_ms": ms, "beam_samples_per_s": 64 * 256 * 16384 / (ms / 1e3)}
    # the same tied beams interpolated from stored complex FFT beams
    beams = bf.beamform_fft(plan, vt, kind=bf.BF_OUT_COMPLEX)
    ms_b = _time_launches(lambda: bf.form_tied_beams(plan, beams, 0, 256, d), 5, warmup=1)
    ex["tied_beams_from_fft_beams"] = {"workload": "same, from the stored complex 4 x 32 FFT beams "
                                                   f"({beams.numel() * 8 / 2**30:.0f} GiB)",
                                       "kernel_ms": ms_b, "beam_samples_per_s": 64 * 256 * 16384 / (ms_b / 1e3),
                                       "hbm_alg_gbs": beams.numel() * 8 / (ms_b / 1e3) / 1e9}
    # the standalone block sum of |B|^2 (bf_accumulate_intensity) over the same stored beams
    z2 = beams.view(beams.shape[0], -1)
    acc_out = torch.empty((z2.shape[0] // 16, z2.shape[1]), dtype=torch.float32, device=dev)
    ms_a = _time_launches(lambda: bf.accumulate_intensity(z2, 16, out=acc_out), 5, warmup=1)
    acc_bytes = z2.numel() * 8 + acc_out.numel() * 4
    acc_rec = {"workload": f"|B|^2 summed over 16 samples of the same stored beams "
                           f"({z2.shape[0]} samples x {z2.shape[1]} series)",
               "kernel_ms": ms_a, "hbm_alg_gbs": acc_bytes / (ms_a / 1e3) / 1e9,
               "hbm_frac": acc_bytes / (ms_a / 1e3) / 1e9 / HBM_PEAK_GBS}
    prng = np.random.default_rng(13)
    for _ in range(2):
        b, c = int(prng.integers(z2.shape[0] // 16)), int(prng.integers(256))
        got = acc_out[b].view(256, 1, 4, 32)[c].cpu().numpy()
        checks.add(acc_rec, "max_rel_power_err_sampled", "fft_rel", got,
                   v=sg.volts(wt, 16 * b, 16, chans=[c]), m_ew=4, m_ns=32, index=(0, 0))
    ex["accumulate_intensity"] = acc_rec
    del beams, z2, acc_out
    plan.close()
    del vt
    torch.cuda.empty_cache()
    ex["larger_lattices"] = _leg(run_larger_lattices, dev, checks)
    ex["serving"] = _leg(run_serving, dev)
    return ex


def run_larger_lattices(dev, checks: OracleChecks) -> dict:
    """FP32, FP16 and FP8 plans on the 4 x 64 and
    4 x 128 lattices at the CHIME channel count and duration, and tied beams
    on the 4 x 256 lattice from voltages (FFT beams through a workspace) and
    from stored complex beams, each with sampled outputs for the oracle."""
    import numpy as np
    import torch

    import paper_1710_08591_amd as bf
    import synthgen as sg
    rec = {}
    for n_ns in (64, 128):
        w = sg.Workload(f"lattice4x{n_ns}_scaled", 4, n_ns, 256, 2, 16384, 4, 2 * n_ns, 16, 8 + n_ns,
                        src_dircos=((0.3, -0.2), (-0.7, 0.5)), src_snr=(10.0, 30.0), dl_lo=0.4, dl_hi=0.8)
        volts = sg.volts(w, backend="torch", device=dev)
        rng = np.random.default_rng(n_ns)
        picks = [(int(rng.integers(w.n_time // 16)), int(rng.integers(w.n_chan)), int(rng.integers(w.n_pol)))
                 for _ in range(2)]
        variants = {}
        for prec, name in ((0, "fp32_fft"), (1, "fp16_mfma"), (2, "fp8_mfma")):
            plan = bf.Plan(n_ew=4, n_ns=n_ns, n_pol=2, n_chan=256, block=16, precision=prec)
            out = torch.empty(plan.out_shape(w.n_time), dtype=torch.float32, device=dev)
            each = []
            ms = _time_launches(lambda: bf.beamform_fft(plan, volts, out=out), 5, warmup=3, each=each)
            variants[name] = {"antenna_samples_per_s": w.antenna_samples / (ms / 1e3), "kernel_ms": ms,
                              "kernel_ms_each": each}
            for b, c, p in picks:
                checks.add(variants[name], "max_rel_power_err_sampled", "fft_rel", out[b, c, p].cpu().numpy(),
                           v=sg.volts(w, b * 16, 16, chans=[c], pols=[p]), m_ew=4, m_ns=2 * n_ns, index=(0, 0, 0))
            plan.close()
            del out
        rec[f"4x{n_ns}"] = {"workload": f"4x{n_ns} lattice, 2 pol, 256 chan, 16384 samples, M_ns = {2 * n_ns}, "
                                        "|B|^2 over 16", "variants": variants}
        del volts
        torch.cuda.empty_cache()
    # tied beams on the 4 x 256 lattice: 64 pointings, 16 channels, 2048 samples
    wt = sg.Workload("tied4x256", 4, 256, 16, 1, 2048, 4, 512, 16, 21,
                     src_dircos=((0.3, -0.2),), src_snr=(20.0,), dl_lo=0.4, dl_hi=0.8)
    vt = sg.volts(wt, backend="torch", device=dev)
    plan = bf.Plan(n_ew=4, n_ns=256, n_chan=16, block=16, d_over_lambda=wt.d_over_lambda())
    dirs = sg.pointings(64, 23)
    d = torch.from_numpy(dirs).to(dev)
    ws = torch.empty(bf.tied_workspace_size(plan, 16, wt.n_time), dtype=torch.uint8, device=dev)
    out = torch.empty((wt.n_time // 16, 16, 1, 64), dtype=torch.float32, device=dev)
    ms_v = _time_launches(lambda: bf.form_tied_beams_v(plan, vt, 0, 16, d, out=out, workspace=ws), 5)
    n_bs = 64 * 16 * wt.n_time
    tv = {"workload": "4x256 lattice, 16 chan, 1 pol, 2048 samples, 64 pointings, |B|^2 over 16; FFT beams "
                      f"({ws.numel() / 2**20:.0f} MiB) through a workspace", "kernel_ms": ms_v,
          "beam_samples_per_s": n_bs / (ms_v / 1e3)}
    dl = wt.d_over_lambda()
    rng = np.random.default_rng(24)
    for b, c in [(0, 0), (int(rng.integers(wt.n_time // 16)), int(rng.integers(16)))]:
        checks.add(tv, "max_rel_power_err_sampled", "tied_rel", out[b, c].cpu().numpy(),
                   v=sg.volts(wt, 16 * b, 16, chans=[c]), dircos=dirs, dl=dl, c=c)
    beams = ws.view(torch.complex64)[: wt.n_time * 16 * 4 * 512].view(wt.n_time, 16, 1, 4, 512)
    bf.beamform_fft(plan, vt, kind=bf.BF_OUT_COMPLEX, out=beams)
    ms_b = _time_launches(lambda: bf.form_tied_beams(plan, beams, 0, 16, d, out=out), 5)
    tb = {"workload": "the same, from the stored complex 4 x 512 FFT beams (FP32 operands as three BF16 terms on the "
                      "matrix cores)",
          "kernel_ms": ms_b, "beam_samples_per_s": n_bs / (ms_b / 1e3),
          "contraction_tflops": n_bs * 8 * 4 * 512 / (ms_b / 1e3) / 1e12}
    for b, c in [(wt.n_time // 16 - 1, 15)]:
        checks.add(tb, "max_rel_power_err_sampled", "tied_rel", out[b, c].cpu().numpy(),
                   v=sg.volts(wt, 16 * b, 16, chans=[c]), dircos=dirs, dl=dl, c=c)
    rec["tied_4x256_from_voltages"] = tv
    rec["tied_4x256_from_fft_beams"] = tb
    plan.close()
    del vt, ws, beams, out
    torch.cuda.empty_cache()
    return rec


def _serve_saturated(srv, reqs) -> dict:
    """Closed loop: every request is submitted as soon as the memory budget
    admits it, so the server always has queued work; the completion rate is
    the highest arrival rate it can sustain for this request mix."""
    import paper_1710_08591_amd as bf
    pending = {}
    i = done = rejected = 0
    beam_samples = 0
    t0 = srv.now()
    while i < len(reqs) or pending:
        while i < len(reqs):
            r = reqs[i]
            st, rid = srv.try_submit(r.dircos, r.chan_lo, r.n_chan, r.n_time)
            if st == bf.BF_OK:
                pending[rid] = r
                i += 1
            elif pending:
                break                                # over budget for now: wait for completions
            else:
                rejected += 1                        # cannot fit even on an idle server
                i += 1
        srv.pump()
        for rid in list(pending):
            st, _ = srv.poll(rid)
            if st == bf.BF_ERR_NOT_READY:
                continue
            r = pending.pop(rid)
            if st == bf.BF_OK:
                done += 1
                beam_samples += r.n_point * r.n_chan * r.n_time
            srv.release(rid)
    span = srv.now() - t0
    return {"requests": len(reqs), "completed": done, "rejected": rejected,
            "requests_per_s": done / span, "beam_samples_per_s": beam_samples / span}


def run_serving(dev, n_req: int = 5200, n_warm: int = 200, rate_hz: float = 200.0, n_sat: int = 1000,
                writer_rate: float = 390625.0, blocks_per_tile: int = 32) -> dict:
    """Open-loop serving of tied-beam requests from a 1 GiB device voltage ring,
    with a writer appending voltages at ``writer_rate`` samples/s meanwhile
    (one sample every 2.56 us, a CHIME-like channelised sample rate)."""
    import numpy as np
    import torch

    import paper_1710_08591_amd as bf
    import synthgen as sg
    w = sg.make_workload("c5")
    plan = bf.Plan(n_ew=4, n_ns=16, n_chan=w.n_chan, n_pol=1, block=16, d_over_lambda=w.d_over_lambda())
    budget = 16 << 30
    srv = bf.Server(plan, ring_samples=w.n_time, hbm_budget=budget, blocks_per_tile=blocks_per_tile,
                    max_tiles_per_launch=8192)
    plan.close()
    step = 4096
    for t0 in range(0, w.n_time, step):          # the writer fills the ring
        src = sg.volts(w, t0, step, backend="torch", device=dev)
        assert srv.advance(step, src) == bf.BF_OK
    torch.cuda.synchronize()
    reqs = sg.request_stream(n_req, seed=5, rate_hz=rate_hz, n_chan_total=w.n_chan)
    pending = {}
    lat = {}
    rejected = 0
    beam_samples = 0
    # a live writer appends voltages to the ring at a fixed sample rate, in
    # chunks, while requests are served; a chunk that would overwrite a leased
    # window is refused and retried (the writer falls behind), and is forced
    # (evicting the lease holders) only once the backlog passes half the ring
    chunk = 1024
    wsrc = sg.volts(w, 0, chunk, backend="torch", device=dev)
    torch.cuda.synchronize()
    writer = {"samples_per_s": writer_rate, "chunk_samples": chunk, "advances": 0, "refused": 0, "forced": 0,
              "max_backlog_samples": 0}
    written = 0
    t_base = srv.now() + 0.05
    i = 0
    while i < len(reqs) or pending:
        now = srv.now()
        backlog = int((now - t_base) * writer_rate) - written if now > t_base else 0
        writer["max_backlog_samples"] = max(writer["max_backlog_samples"], backlog)
        if backlog >= chunk:
            force = backlog > w.n_time // 2
            st = srv.advance(chunk, wsrc, force=force)
            if st == bf.BF_OK:
                written += chunk
                writer["advances"] += 1
                writer["forced"] += int(force)
            else:
                writer["refused"] += 1
        while i < len(reqs) and t_base + reqs[i].arrival_s <= now:
            r = reqs[i]
            st, rid = srv.try_submit(r.dircos, r.chan_lo, r.n_chan, r.n_time, arrival=t_base + r.arrival_s)
            if st == bf.BF_OK:
                pending[rid] = r
            else:
                rejected += 1
            i += 1
        srv.pump()
        for rid in list(pending):
            st, l = srv.poll(rid)
            if st == bf.BF_ERR_NOT_READY:
                continue
            r = pending.pop(rid)
            if st == bf.BF_OK:
                lat[r.rid] = l
                if r.rid >= n_warm:
                    beam_samples += r.n_point * r.n_chan * r.n_time
            srv.release(rid)
    t_end = srv.now()
    st = srv.stats()
    writer["achieved_samples_per_s"] = written / (t_end - t_base)
    writer["evicted_requests"] = st.get("evicted")
    sat = _serve_saturated(srv, sg.request_stream(n_sat, seed=6, rate_hz=rate_hz, n_chan_total=w.n_chan))
    srv.close()
    measured = [lat[k] for k in sorted(lat) if k >= n_warm]
    arr = [t_base + r.arrival_s for r in reqs if r.rid >= n_warm]
    span = t_end - min(arr)
    ms = np.array(measured) * 1e3
    return {"workload": "tied-beam requests on a 4x16 lattice ring (65536 samples x 256 chan x 1 pol, 1 GiB); "
                        "Poisson 200/s; pointings, duration (1024-65536) and channel count (8-256) log-uniform; "
                        "a live writer appends voltages at one sample per 2.56 us meanwhile",
            "requests": n_req, "warmup_requests": n_warm, "rejected": rejected,
            "p50_ms": float(np.percentile(ms, 50)), "p99_ms": float(np.percentile(ms, 99)),
            "mean_ms": float(ms.mean()), "max_ms": float(ms.max()),
            "requests_per_s": len(measured) / span, "beam_samples_per_s": beam_samples / span,
            "launches": st["launches"], "tiles": st["tiles_done"], "hbm_budget_bytes": budget,
            "live_writer": writer,
            "max_sustainable": dict(sat, workload="closed loop over the same request mix (seed 6): "
                                                  "each request submitted as soon as memory admits it")}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--skip-extras", action="store_true", help="only the headline FP32 measurement")
    ap.add_argument("--skip-cpu", action="store_true", help="no CPU oracle baseline")
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    args = ap.parse_args()
    if args.gpus != 1:
        print(json.dumps({"error": "this benchmark runs on one GPU; the path shards by frequency channel "
                                   "across GPUs but no multi-GPU run is provided", "n_gpus": args.gpus}))
        sys.exit(2)

    import numpy as np
    import torch

    import paper_1710_08591_amd as bf
    import synthgen as sg

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    w = sg.make_workload("c2")
    plan = bf.Plan(n_ew=w.n_ew, n_ns=w.n_ns, m_ew=w.m_ew, m_ns=w.m_ns, n_pol=w.n_pol, n_chan=w.n_chan,
                   block=w.block, ns_select=w.ns_select(), d_over_lambda=w.d_over_lambda())
    tg = time.perf_counter()
    volts = sg.volts(w, backend="torch", device=dev)
    out = torch.empty(plan.out_shape(w.n_time), dtype=torch.float32, device=dev)
    torch.cuda.synchronize()
    gen_s = time.perf_counter() - tg
    stream = torch.cuda.current_stream()

    for _ in range(args.warmup):
        bf.beamform_fft(plan, volts, out=out)
    torch.cuda.synchronize()

    # Each step is exactly one kernel launch on `stream`; events bracket each
    # launch so the average kernel duration is measured live.
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
    torch.cuda.synchronize()
    with _no_gc():
        t_start = time.perf_counter()
        for i in range(args.steps):
            ev[i][0].record(stream)
            bf.beamform_fft(plan, volts, out=out)
            ev[i][1].record(stream)
        torch.cuda.synchronize()
        wall = time.perf_counter() - t_start
    kern_ms = [a.elapsed_time(b) for a, b in ev]
    ms_avg = float(np.mean(kern_ms))
    ms_step = wall * 1000.0 / args.steps

    ant_samples = w.antenna_samples
    value = ant_samples / (ms_step / 1000.0)
    frames = w.n_time * w.n_chan * w.n_pol
    flops = frames * flops_per_frame(w.n_ns, w.m_ns, w.keep)
    achieved_tflops = flops / (ms_avg / 1000.0) / 1e12
    mfma_tops = lag_products(frames) / (ms_avg / 1000.0) / 1e12
    in_bytes = w.n_time * w.n_chan * w.n_pol * w.frame_bytes
    out_bytes = out.numel() * 4
    alg_bytes = in_bytes + out_bytes
    src_hash = kernel_source_hash("k_lag.hip", "dev_bytes.h")
    prof = counters_from_profile("traffic_lag_chime.json", src_hash)
    traffic = prof.get("hbm_bytes_per_launch")
    # vector instructions issued per SIMD and clock cycle (counted
    # instructions over the live launch time, at the peak clock)
    valu = prof.get("sq_insts_valu_per_launch")
    valu_rate = (valu / (N_SIMD * CLOCK_HZ * ms_avg / 1000.0)) if valu else None

    rec = {
        "metric": METRIC,
        "value": value,
        "unit": "antenna-samples/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_step,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": "chime_fp32: 4x256 lattice, 2 pol, 256 chan, 16384 samples int4+4, "
                               "N-S zero-padded to 512, clamp to 256 N-S beams, |B|^2 over 16 samples",
                   "lattice": [4, 256], "n_pol": 2, "n_chan": 256, "n_time": 16384, "m_ns": 512,
                   "n_ns_keep": 256, "block": 16, "precision": "fp32"},
        # what the kernel executes: int8 matrix products (the FFT's nominal flops beside them, of a transform
        # per sample that does not run)
        "roofline": {"bound": "mfma", "achieved": mfma_tops, "peak": INT8_MFMA_PEAK_TOPS,
                     "unit": "TOP/s int8", "frac": mfma_tops / INT8_MFMA_PEAK_TOPS,
                     "traffic": traffic,
                     "kernel": "k_lag<256> (stacked visibilities: exact int8 products, FP64 transforms per block)",
                     "nominal_fft_tflops": achieved_tflops,
                     "nominal_fft_frac_of_fp32_vector_peak": achieved_tflops / FP32_VECTOR_PEAK_TFLOPS,
                     "kernel_ms": ms_avg,
                     "kernel_ms_p10_p50_p90": [float(np.percentile(kern_ms, q)) for q in (10, 50, 90)],
                     "valu_insts_per_launch": valu,
                     "valu_insts_per_simd_cycle": valu_rate,
                     "flop_per_antenna_sample": flops / ant_samples,
                     "hbm_alg_bytes": alg_bytes,
                     "hbm_alg_gbs": alg_bytes / (ms_avg / 1000.0) / 1e9,
                     "hbm_frac": alg_bytes / (ms_avg / 1000.0) / 1e9 / HBM_PEAK_GBS},
        "generation_s": gen_s,
    }
    # sampled slices of the headline output; the oracle leg fills in the error
    checks = OracleChecks()
    rec["parity"] = {"reference": "FP64 oracle (direct phased sums): every channel and pol of the first and the "
                                  "last block of the timed output (each channel's own clamp table) and 4 random "
                                  "(block, channel, pol) slices, all 1024 kept beams each",
                     "tolerance": 1e-5}
    checks.add_blocks(rec["parity"], "max_rel_power_err_sampled", out, w)
    prng = np.random.default_rng(11)
    sel = w.ns_select()
    for _ in range(4):
        blk, c, p = (int(prng.integers(w.n_time // w.block)), int(prng.integers(w.n_chan)),
                     int(prng.integers(w.n_pol)))
        checks.add(rec["parity"], "max_rel_power_err_sampled", "fft_rel", out[blk, c, p].cpu().numpy(),
                   v=sg.volts(w, blk * w.block, w.block, chans=[c], pols=[p]), m_ew=w.m_ew, m_ns=w.m_ns,
                   index=(0, 0, 0), sel=sel[c])

    chime_mixed = chime_regrid = library_fft = chime_coadding = None
    if not args.skip_extras:
        chime_mixed = _leg(run_chime_mixed, dev, w, volts, ms_avg, checks)
        del out
        torch.cuda.empty_cache()
        chime_coadding = _leg(run_chime_coadding, dev, w, volts, ms_avg, checks)
        torch.cuda.empty_cache()
        chime_regrid = _leg(run_chime_regrid, dev, w, volts, ms_avg, checks)
        torch.cuda.empty_cache()
        library_fft = _leg(run_library_fft_comparator, dev, w, volts, plan, ms_avg)
        torch.cuda.empty_cache()
    else:
        del out
    del volts
    plan.close()
    torch.cuda.empty_cache()
    if not args.skip_extras:
        rec["extras"] = {"chime_fp16_mfma": chime_mixed, "chime_regrid": chime_regrid,
                         "chime_cyclic_coadding": chime_coadding, "library_fft_comparator": library_fft}
        rec["extras"].update(_leg(run_extras, dev, checks))
        torch.cuda.empty_cache()
    if not args.skip_cpu:
        rec["cpu_baseline"] = _leg(cpu_baseline, args.cpu_seconds, checks)
    print(json.dumps(rec))


if __name__ == "__main__":
    main()
