"""Performance cases: the calls that a program using this beamformer makes, at the sizes of its configurations.

A case is a dict of plain values with a "kind":
  intensity  voltages -> FFT-beam intensities (beamform_fft): the hot path of every backend
  chain      voltages -> unclamped intensities -> regridded (achromatic) beams, on one or both axes
  localize   stored intensities -> source positions (a search backend's triggers)
  stored     voltages -> complex FFT beams -> tied-array beams and beam powers of the stored beams
  tied       voltages -> tied-array beam intensities at arbitrary pointings (a pulsar or follow-up backend)
  serve      a burst of tied-beam requests through the server, from a filled ring of voltages

Voltages are int4+4 samples: Gaussian noise (sigma 2) plus a few sources of
beam-level SNR 5 to 50, rounded and clipped to [-7, 7].
"""
import math

import numpy as np
import torch

import paper_1710_08591_amd as bf

PREC = {"fp32": bf.BF_PREC_FP32, "fp16": bf.BF_PREC_FP16_MFMA, "fp8": bf.BF_PREC_FP8_MFMA}
DEV = "cuda"


# ---- the cases -------------------------------------------------------------
def _intensity(n_ns, n_chan, n_pol, block, n_blk, prec="fp32", weights="none", keep=0, pol_sum=False, m_ew=4, m_ns=0):
    """keep 0: every N-S beam; m_ns 0: zero-padded to 2 n_ns; weights: none, window (real) or gains (complex)."""
    return {"kind": "intensity", "n_ns": n_ns, "n_chan": n_chan, "n_pol": n_pol, "block": block, "n_blk": n_blk,
            "prec": prec, "weights": weights, "keep": keep, "pol_sum": pol_sum, "m_ew": m_ew, "m_ns": m_ns}


def _chain(n_ns, n_chan, n_pol, block, n_blk, n_target, n_taps=0, m_ew=4):
    """m_ew 8: exact 2-D pointings; else N-S steering angles, dense (n_taps 0) or compact kernels."""
    return {"kind": "chain", "n_ns": n_ns, "n_chan": n_chan, "n_pol": n_pol, "block": block, "n_blk": n_blk,
            "n_target": n_target, "n_taps": n_taps, "m_ew": m_ew}


def _localize(n_ns, n_chan, n_pol, n_blk):
    return {"kind": "localize", "n_ns": n_ns, "n_chan": n_chan, "n_pol": n_pol, "n_blk": n_blk}


def _tied(kind, n_ns, n_chan, n_pol, block, n_blk, n_point, window=False, pol_sum=False):
    return {"kind": kind, "n_ns": n_ns, "n_chan": n_chan, "n_pol": n_pol, "block": block, "n_blk": n_blk,
            "n_point": n_point, "window": window, "pol_sum": pol_sum}


def _serve(n_chan, ring, n_req, mix):
    """mix: seed of the request sizes (pointings 1-256, samples 1024 to the ring, channels 8 to n_chan)."""
    return {"kind": "serve", "n_chan": n_chan, "ring": ring, "n_req": n_req, "mix": mix}


def listed():
    return [
        # the smallest configuration, one call: a test bench or one coarse channel of a small array; latency counts
        dict(_intensity(16, 1, 1, 16, 64), name="tiny_fp32"),
        # the same array at a full band and two polarisations, matrix-core FP8 plan
        dict(_intensity(16, 256, 2, 16, 1024, prec="fp8"), name="lattice16_fp8"),
        # a mid-size array searched in total intensity (summed polarisations), odd channel count and a 20-sample block
        dict(_intensity(64, 93, 2, 20, 200, pol_sum=True), name="lattice64_fp32_stokes_i"),
        # CHIME-shaped fast-radio-burst backend: 2048 antennas, 1024 formed beams per channel; the headline workload
        dict(_intensity(256, 256, 2, 16, 1024, keep=256), name="chime_fp32"),
        # the same backend on an FP16 matrix-core plan, a quarter of the length
        dict(_intensity(256, 256, 2, 16, 256, prec="fp16", keep=256), name="chime_fp16"),
        # with sculpted (apodised) beams
        dict(_intensity(256, 256, 2, 16, 256, weights="window", keep=256), name="chime_fp32_window"),
        # with per-antenna calibration gains
        dict(_intensity(256, 256, 2, 16, 128, weights="gains", keep=256), name="chime_fp32_gains"),
        # exact 2-D pointings from intensities: E-W axis padded, then regridded
        dict(_chain(256, 64, 2, 16, 128, 256, m_ew=8), name="chime_pointings_2d"),
        # source localisation on a stored block of beams
        dict(_localize(256, 256, 2, 64), name="chime_localize"),
        # complex beams kept, then pointed and integrated (a baseband recorder's replay)
        dict(_tied("stored", 64, 32, 2, 16, 128, 48), name="stored_beams_lattice64"),
        # tied beams straight from voltages: 64 pointings over the full band of the small array
        dict(_tied("tied", 16, 256, 1, 16, 1024, 64), name="tied64_lattice16"),
        # the tied-beam server: a burst of requests of uneven size against a full ring
        dict(_serve(256, 65536, 24, 5), name="serve_burst"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["intensity"] * 6 + ["chain", "localize", "stored", "tied", "tied", "serve"])
    n_ns = rng.choice([16, 32, 64, 128, 256])
    n_pol = rng.choice([1, 2])
    n_chan = _log(rng, 1, 256)
    if kind == "intensity":
        block = rng.choice([16, 16, 16, 32, 48, 64, 4 * rng.randint(1, 40)])
        prec, weights, m_ew, m_ns = "fp32", "none", 4, 0
        option = rng.choice(["fp32", "fp32", "fp32", "fp16", "fp16", "fp8", "window", "window16", "gains", "ew8", "coadd"])
        if option in ("fp16", "fp8", "window16"):
            prec, block = ("fp8" if option == "fp8" else "fp16"), 16 * rng.choice([1, 1, 2, 3, 5])
        if option in ("window", "window16"):
            weights = "window"
        if option == "gains":
            weights = "gains"
        if option == "ew8":
            m_ew = 8
        if option == "coadd":
            n_ns = rng.choice([64, 128, 256])
            m_ns = n_ns // rng.choice([2, 4])
        frames = _log(rng, 64, 1 << 21)               # (sample, channel, polarisation) frames
        n_blk = max(1, min(4096, frames // (block * n_chan * n_pol)))
        keep = 0 if option == "coadd" or rng.random() < 0.5 else rng.randint(1, 2 * n_ns)
        return _intensity(n_ns, n_chan, n_pol, block, n_blk, prec, weights, keep, rng.random() < 0.3, m_ew, m_ns)
    frames = _log(rng, 256, 1 << 19)
    block = rng.choice([16, 16, 32, 48])
    n_blk = max(1, min(2048, frames // (block * n_chan * n_pol)))
    if kind == "chain":
        m_ew = rng.choice([4, 8])
        return _chain(n_ns, n_chan, n_pol, block, n_blk, _log(rng, 8, 400), rng.choice([0, 0, 5]) if m_ew == 4 else 0, m_ew)
    if kind == "localize":
        return _localize(n_ns, n_chan, n_pol, n_blk)
    if kind in ("stored", "tied"):
        return _tied(kind, n_ns, n_chan, n_pol, block, n_blk, _log(rng, 1, 256), rng.random() < 0.3, rng.random() < 0.3)
    return _serve(rng.choice([16, 64, 256]), 16384, rng.randint(1, 24), rng.randrange(1 << 20))


# ---- inputs ----------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _volts(seed, n_time, n_chan, n_pol, n_ns, n_src=3):
    """uint8 [t][chan][pol][n_ns][4]: noise and point sources, digitised to int4+4."""
    g = _gen(seed)
    r = np.random.default_rng(seed)
    a_ns = torch.arange(n_ns, device=DEV, dtype=torch.float64)[:, None]
    a_ew = torch.arange(4, device=DEV, dtype=torch.float64)[None, :]
    sources = []
    for _ in range(n_src):
        snr = float(r.uniform(5.0, 50.0))
        phi = 2 * math.pi * (a_ns * float(r.uniform(-0.5, 0.5)) + a_ew * float(r.uniform(-0.5, 0.5)))
        sources.append((2.0 * snr / math.sqrt(4 * n_ns), phi.cos().float(), phi.sin().float()))
    out = torch.empty((n_time, n_chan, n_pol, n_ns, 4), dtype=torch.uint8, device=DEV)
    step = max(1, (1 << 26) // (n_chan * n_pol * n_ns * 4))
    for t0 in range(0, n_time, step):
        o = out[t0:t0 + step]
        parts = [torch.randn(o.shape, device=DEV, generator=g).mul_(2.0) for _ in range(2)]
        for amp, c, s in sources:
            zr, zi = (torch.randn(o.shape[:3] + (1, 1), device=DEV, generator=g).mul_(amp * 0.7071) for _ in range(2))
            parts[0].addcmul_(zr, c).addcmul_(zi, s, value=-1.0)
            parts[1].addcmul_(zr, s).addcmul_(zi, c)
        re, im = (p.round_().clamp_(-7, 7).to(torch.int8).view(torch.uint8) for p in parts)
        torch.bitwise_or(re << 4, im & 15, out=o)
    return out


def _window(n_ns):
    """Gaussian taper, width 0.4 of the aperture on both axes."""
    def h(n):
        a = np.arange(n)
        return np.exp(-0.5 * ((a - (n - 1) / 2) / (0.4 * n)) ** 2)
    return np.outer(h(n_ns), h(4)).astype(np.float32)


def _weights(case, seed):
    """Host weights [n_ns][4] (float32 window or complex64 gains) or None."""
    if case.get("window") or case.get("weights") == "window":
        return _window(case["n_ns"])
    if case.get("weights") == "gains":
        r = np.random.default_rng(seed + 77)
        shape = (case["n_ns"], 4)
        return (np.exp(0.1 * r.standard_normal(shape)) * np.exp(1j * r.uniform(-np.pi, np.pi, shape))).astype(np.complex64)
    return None


def _dl(n_chan):
    return np.repeat(np.linspace(0.4, 0.8, n_chan)[:, None], 2, axis=1)


def _select(case):
    """The per-channel clamp table: the FFT beams nearest a fixed grid of sin(theta)."""
    keep, m = case.get("keep", 0), case.get("m_ns") or 2 * case["n_ns"]
    if not keep:
        return None
    st = -1 + (np.arange(keep) + 0.5) * 2 / keep
    return (np.rint(st[None, :] * _dl(case["n_chan"])[:, 1:] * m).astype(np.int64) % m).astype(np.int32)


def _plan(case, prec="fp32", sel=None):
    return bf.Plan(n_ew=4, n_ns=case["n_ns"], m_ew=case.get("m_ew", 4), m_ns=case.get("m_ns") or None,
                   n_pol=case["n_pol"], n_chan=case["n_chan"], block=case.get("block", 16), ns_select=sel,
                   pol_sum=case.get("pol_sum", False), precision=PREC[prec], d_over_lambda=_dl(case["n_chan"]))


def _pointings(seed, n):
    return np.random.default_rng(seed + 5).uniform(-0.95, 0.95, (n, 2))


def _targets(case):
    return np.linspace(-0.95, 0.95, case["n_target"])


def _rows(case, seed):
    """Stored intensities [blk][chan][pol][4][m]: noise powers of 16-sample blocks and one source per row."""
    g, n, m = _gen(seed), case["n_ns"], 2 * case["n_ns"]
    shape = (case["n_blk"], case["n_chan"], case["n_pol"], 4, m)
    x = torch.empty(shape, device=DEV)
    x.normal_(128.0, 32.0, generator=g).clamp_(min=8.0)
    y = torch.rand(shape[:-1] + (1,), device=DEV, generator=g)
    u = y - torch.arange(m, device=DEV) / m
    d = torch.sin(math.pi * n * u) / (n * torch.sin(math.pi * u)).abs().clamp_(min=1e-6)
    return x.addcmul_(d, d, value=20000.0)


def _requests(case):
    r = np.random.default_rng(case["mix"])
    out = []
    for _ in range(case["n_req"]):
        n_time = 16 * int(math.exp(r.uniform(math.log(64), math.log(case["ring"] // 16))))
        n_ch = int(round(math.exp(r.uniform(math.log(8), math.log(case["n_chan"])))))
        n_pt = int(round(math.exp(r.uniform(0, math.log(256)))))
        out.append((r.uniform(-0.95, 0.95, (n_pt, 2)), int(r.integers(0, case["n_chan"] - n_ch + 1)), n_ch, n_time))
    return out


# ---- the passes --------------------------------------------------------------
def prepare(case, seed):
    s = {"case": case}
    kind = case["kind"]
    if kind == "localize":
        s["plan"] = _plan(case)
        s["rows"] = _rows(case, seed)
        return s
    if kind == "serve":
        plan = bf.Plan(n_ew=4, n_ns=16, n_chan=case["n_chan"], n_pol=1, block=16, d_over_lambda=_dl(case["n_chan"]))
        s["server"] = bf.Server(plan, ring_samples=case["ring"], hbm_budget=6 << 30)
        plan.close()
        v = _volts(seed, case["ring"], case["n_chan"], 1, 16)
        if s["server"].advance(case["ring"], v) != bf.BF_OK:
            raise RuntimeError("the ring could not be filled")
        torch.cuda.synchronize()
        s["requests"] = _requests(case)
        return s
    w = _weights(case, seed)
    s["volts"] = _volts(seed, case["n_blk"] * case["block"], case["n_chan"], case["n_pol"], case["n_ns"])
    s["w"] = None if w is None else torch.from_numpy(w).to(DEV)
    if kind == "intensity":
        s["plan"] = _plan(case, case["prec"], _select(case))
    else:
        s["plan"] = _plan(case)
    n_time = case["n_blk"] * case["block"]
    if kind in ("intensity", "chain"):
        s["out"] = torch.empty(s["plan"].out_shape(n_time), device=DEV)
    if kind == "chain":
        s["regrid"] = (bf.Regrid2D(s["plan"], _pointings(seed, case["n_target"])) if case["m_ew"] == 8
                       else bf.Regrid(s["plan"], _targets(case), n_taps=case["n_taps"]))
    if kind in ("stored", "tied"):
        s["dircos"] = torch.from_numpy(_pointings(seed, case["n_point"])).to(DEV)
    if kind == "stored":
        s["beams"] = torch.empty(s["plan"].out_shape(n_time, bf.BF_OUT_COMPLEX), dtype=torch.complex64, device=DEV)
    return s


def run(s):
    case, kind = s["case"], s["case"]["kind"]
    if kind == "intensity":
        if case["weights"] == "gains":
            return bf.beamform_fft(s["plan"], s["volts"], gains=s["w"], out=s["out"])
        return bf.beamform_fft(s["plan"], s["volts"], s["w"], out=s["out"])
    if kind == "chain":
        i = bf.beamform_fft(s["plan"], s["volts"], out=s["out"])
        return [i, s["regrid"](i)]
    if kind == "localize":
        return list(bf.localize(s["plan"], s["rows"]))
    if kind == "stored":
        b = bf.beamform_fft(s["plan"], s["volts"], s["w"], kind=bf.BF_OUT_COMPLEX, out=s["beams"])
        return [b, bf.form_tied_beams(s["plan"], b, 0, case["n_chan"], s["dircos"]),
                bf.accumulate_intensity(b.view(b.shape[0], -1), case["block"])]
    if kind == "tied":
        return bf.form_tied_beams_v(s["plan"], s["volts"], 0, case["n_chan"], s["dircos"], taper=s["w"])
    srv = s["server"]
    ids = [srv.submit(*q) for q in s["requests"]]
    outs = [None] * len(ids)
    left = set(range(len(ids)))
    while left:
        srv.pump()
        for k in sorted(left):
            st, _ = srv.poll(ids[k])
            if st == bf.BF_ERR_NOT_READY:
                continue
            if st != bf.BF_OK:
                raise RuntimeError(f"request {k}: status {st}")
            outs[k] = srv.result(ids[k])
            left.discard(k)
    torch.cuda.current_stream().synchronize()      # the copies have left the pool before it is given back
    for i in ids:
        srv.release(i)
    return outs


# ---- what a pass cannot do without ---------------------------------------------
def work(case):
    kind, n = case["kind"], case.get("n_ns", 16)
    m = case.get("m_ns") or 2 * n
    m_ew = case.get("m_ew", 4)
    if kind == "serve":
        nbytes = flops = 0.0
        for d, _, n_ch, n_time in _requests(case):
            frames = n_time * n_ch
            nbytes += frames * 64 + frames / 16 * len(d) * 4
            flops += frames * (4 * 5 * 32 * 5 + 4 * len(d))     # FFT beams, one accumulated power per pointing
        return {"bytes": nbytes, "flops": flops}
    groups = case["n_blk"] * case["n_chan"] * (1 if case.get("pol_sum") else case["n_pol"])
    if kind == "localize":
        return {"bytes": groups * 4 * (m * 4 + 12), "flops": groups * 4 * 6 * 10 * 20}
    frames = case["n_blk"] * case["block"] * case["n_chan"] * case["n_pol"]
    fft = m_ew * 5 * m * math.log2(m) + 16 * n                 # one frame's transform
    if kind in ("intensity", "chain"):
        keep = case.get("keep") or m
        nbytes, flops = frames * 4 * n + groups * m_ew * keep * 4, frames * (fft + 4 * m_ew * keep)
        if kind == "chain":
            rows = groups * m_ew
            nbytes += rows * m * 4 + (groups if m_ew == 8 else rows) * case["n_target"] * 4
            flops += rows * case["n_target"] * 2 * (case["n_taps"] or m)
        return {"bytes": nbytes, "flops": flops}
    if kind == "stored":
        nbytes = frames * (4 * n + 3 * 4 * m * 8) + groups * case["n_point"] * 4
        return {"bytes": nbytes + case["n_blk"] * case["n_chan"] * case["n_pol"] * 4 * m * 4,
                "flops": frames * (fft + 4 * 4 * m + case["n_point"] * (8 * 4 * m + 4))}
    return {"bytes": frames * 4 * n + groups * case["n_point"] * 4, "flops": frames * (fft + 4 * case["n_point"])}


# ---- the same in 64 bits ---------------------------------------------------------
def _decode(v):
    b = v.view(torch.int8)
    lo = b << 4
    return torch.complex((b >> 4).double(), (lo >> 4).double())


def _exact_beams(x, w, m_ew, m_ns):
    """Complex FFT beams [t][chan][pol][m_ew][m_ns] of decoded voltages."""
    n_ns = x.shape[3]
    if w is not None:
        x = x * w
    if m_ns < n_ns:
        x = x.reshape(x.shape[:3] + (n_ns // m_ns, m_ns, 4)).sum(3)
    x = torch.fft.fft(torch.fft.fft(x, n=m_ns, dim=3), n=m_ew, dim=4)
    return x.transpose(3, 4) / math.sqrt(4 * n_ns)


def _power(x):
    return x.real.square() + x.imag.square()


def _blocks(case, per_frame, fn, v):
    """fn over pieces of whole blocks of v, joined."""
    block = case["block"]
    step = block * max(1, int((1 << 27) // (per_frame * v.shape[1] * v.shape[2] * block)))
    return torch.cat([fn(v[t:t + step]) for t in range(0, v.shape[0], step)])


def _sum_blocks(p, block, pol_sum):
    p = p.reshape((p.shape[0] // block, block) + p.shape[1:]).sum(1)
    return p.sum(2) if pol_sum else p


def _exact_intensity(case, v, w):
    m_ew, m_ns = case.get("m_ew", 4), case.get("m_ns") or 2 * case["n_ns"]
    sel = _select(case)
    idx = None if sel is None else torch.from_numpy(sel.astype(np.int64)).to(v.device)

    def part(x):
        p = _sum_blocks(_power(_exact_beams(_decode(x), w, m_ew, m_ns)), case["block"], case.get("pol_sum", False))
        if idx is None:
            return p
        at = idx.view((1, idx.shape[0]) + (1,) * (p.dim() - 3) + (-1,))
        return p.gather(-1, at.expand(p.shape[:-1] + (idx.shape[1],)))
    return _blocks(case, m_ew * m_ns, part, v)


def _steer(n_ns, dl, d, w):
    """Pointed weights [chan][n_ns * 4][point] of direction cosines d, complex128."""
    a_ns = torch.arange(n_ns, device=DEV, dtype=torch.float64)
    a_ew = torch.arange(4, device=DEV, dtype=torch.float64)
    y_ew, y_ns = dl[:, 0:1] * d[:, 0], dl[:, 1:2] * d[:, 1]                 # [chan][point]
    ph = a_ns[:, None, None, None] * y_ns + a_ew[:, None, None] * y_ew       # [ns][ew][chan][point]
    wt = torch.polar(torch.ones_like(ph), -2 * math.pi * ph) / math.sqrt(4 * n_ns)
    if w is not None:
        wt = wt * w[:, :, None, None]
    return wt.reshape(n_ns * 4, dl.shape[0], -1).transpose(0, 1).contiguous()


def _exact_tied(case, v, w, d):
    """Direct phased sums, channel by channel: [blk][chan]([pol])[point]."""
    n_ns, block, n_pol = v.shape[3], case["block"], v.shape[2]
    dl = torch.from_numpy(_dl(case["n_chan"])[case.get("lo", 0):][:v.shape[1]]).to(DEV)
    wt = _steer(n_ns, dl, d, w)
    out = torch.empty((v.shape[0] // block, v.shape[1], n_pol, d.shape[0]), dtype=torch.float64, device=DEV)
    step = block * max(1, (1 << 22) // (block * n_pol * max(d.shape[0], n_ns * 4)))
    for c in range(v.shape[1]):
        for t in range(0, v.shape[0], step):
            x = _decode(v[t:t + step, c]).reshape(-1, n_ns * 4)
            p = _power(x @ wt[c]).reshape(-1, block, n_pol, d.shape[0]).sum(1)
            out[t // block:t // block + p.shape[0], c] = p
    return out.sum(2) if case.get("pol_sum") else out


def _kernel(n, m, y):
    """Regridding weights (1/m) sin((2n-1) pi u) / sin(pi u) of y [...] onto the m beams: [...][m]."""
    u = y[..., None] - torch.arange(m, device=y.device, dtype=torch.float64) / m
    s = torch.sin(math.pi * u)
    near = s.abs() < 1e-12
    return torch.where(near, torch.full_like(s, 2 * n - 1.0), torch.sin((2 * n - 1) * math.pi * u)
                       / torch.where(near, torch.ones_like(s), s)) / m


def _exact_chain(case, seed, v):
    n, m = case["n_ns"], 2 * case["n_ns"]
    full = _exact_intensity(case, v, None)
    dl = torch.from_numpy(_dl(case["n_chan"])).to(DEV)
    shape = full.shape[:4] + (case["n_target"],) if case["m_ew"] == 4 else full.shape[:3] + (case["n_target"],)
    out = torch.empty(shape, dtype=torch.float64, device=DEV)
    pts = torch.from_numpy(_pointings(seed, case["n_target"])).to(DEV)
    st = torch.from_numpy(_targets(case)).to(DEV)
    for c in range(case["n_chan"]):
        y = dl[c, 1] * (pts[:, 1] if case["m_ew"] == 8 else st)
        w = _kernel(n, m, y)
        k = case["n_taps"]
        if k:
            first = torch.round(y * m).long() - (k - 1) // 2
            near = torch.zeros_like(w).scatter_(1, (first[:, None] + torch.arange(k, device=DEV)) % m, 1.0)
            w = w * near
        o = full[:, c] @ w.t()
        if case["m_ew"] == 8:
            o = (o * _kernel(4, 8, dl[c, 0] * pts[:, 0]).t()).sum(-2)
        out[:, c] = o
    return [full, out]


def _exact_localize(case, rows, n_window=10, n_iter=6):
    n, m = case["n_ns"], 2 * case["n_ns"]
    dl = torch.from_numpy(_dl(case["n_chan"])[:, 1]).to(DEV)
    lag = torch.arange(1, n, device=DEV, dtype=torch.float64)
    moi = float((2 * lag * lag * (n - lag)).sum())

    def part(x):
        b, top = x.max(-1)
        top = x.argmax(-1)
        idx = (top[..., None] - (n_window - 1) // 2 + torch.arange(n_window, device=DEV)) % m
        v = x.gather(-1, idx).double().reshape(-1, n_window)
        idx = idx.reshape(-1, n_window).double()
        y0 = top.reshape(-1).double() / m
        y, live = y0.clone(), torch.ones_like(y0, dtype=torch.bool)

        def power(y):
            u = 2 * math.pi * (y[:, None] - idx / m)
            d, s = torch.ones_like(u), torch.zeros_like(u)
            z = torch.polar(torch.ones_like(u), u)
            zk = torch.ones_like(z)
            for k in range(1, n):
                zk = zk * z
                d += 2 * zk.real
                s -= 4 * math.pi * k * zk.imag
            return (v * d).sum(-1) / m, (v * s).sum(-1) / m
        for _ in range(n_iter):
            p, dp = power(y)
            new = y + n * n * dp / (4 * math.pi ** 2 * moi * p)
            live = live & (p > 0) & ((new - y0).abs() <= 1.0 / m)
            y = torch.where(live, new, y)
        p, _ = power(y)
        y = y - torch.floor(y + 0.5)
        return (y.reshape(b.shape) / dl[None, :, None, None]), p.reshape(b.shape)
    step = max(1, (1 << 18) // (4 * rows.shape[1] * rows.shape[2]))
    got = [part(rows[t:t + step]) for t in range(0, rows.shape[0], step)]
    return [torch.cat([g[0] for g in got]), torch.cat([g[1] for g in got])]


def exact(case, seed):
    kind = case["kind"]
    if kind == "localize":
        return _exact_localize(case, _rows(case, seed))
    if kind == "serve":
        v = _volts(seed, case["ring"], case["n_chan"], 1, 16)
        outs = []
        for d, lo, n_ch, n_time in _requests(case):
            c = {"n_chan": case["n_chan"], "block": 16, "lo": lo}
            outs.append(_exact_tied(c, v[-n_time:, lo:lo + n_ch], None, torch.from_numpy(d).to(DEV)))
        return outs
    w = _weights(case, seed)
    w = None if w is None else torch.from_numpy(w).to(DEV).to(torch.complex128)
    v = _volts(seed, case["n_blk"] * case["block"], case["n_chan"], case["n_pol"], case["n_ns"])
    if kind == "intensity":
        return _exact_intensity(case, v, w)
    if kind == "chain":
        return _exact_chain(case, seed, v)
    d = None if kind not in ("tied", "stored") else torch.from_numpy(_pointings(seed, case["n_point"])).to(DEV)
    tied = _exact_tied(case, v, w, d)
    if kind == "tied":
        return tied
    m = 2 * case["n_ns"]
    b = _blocks(case, 4 * m, lambda x: _exact_beams(_decode(x), w, 4, m), v)
    p = _power(b).reshape(case["n_blk"], case["block"], -1).sum(1)
    return [b, tied, p]
