"""Performance cases of the correlator: what its users have it do, through its public entry points.

Each case is a dict of plain values with a "kind"; the kinds are

  fx        one call of the F+X (any input word, filter, antenna count, precision),
  plan      several arrays together through a batched plan,
  calibrate one interval's MAD flags, delay/phase solve and correction,
  mad       MAD flags of a whole observation's visibilities,
  flagger   normalisation and logits of the learned flagger (inference),
  train     one training step of the learned flagger,
  image     dirty image, synthesized beam and CLEAN.

prepare() makes the inputs on the GPU from a seed, run() is one pass, exact()
the same results in 64 bits by plain torch.
"""

from __future__ import annotations

import math

import torch

import paper_2604_20640_amd as qc

FS_HZ = 1.0e9            # sampling rate that turns channel numbers into Hz
C_LIGHT = 299792458.0
COMPLEX_WORDS = ("ci8", "ci16")
WORD_BYTES = {"i8": 1, "i16": 2, "ci8": 2, "ci16": 4}


# ---- the cases ------------------------------------------------------------------------------

def _fx(name, n_ant, n_fft, n_spec, per_dump, **kw):
    c = {"kind": "fx", "n_ant": n_ant, "n_fft": n_fft, "n_spec": n_spec, "per_dump": per_dump,
         "n_taps": 4, "window": "hann", "word": "i8", "x_prec": "f32", "carry": False}
    c.update(kw)
    return {"name": name, **c} if name else c


def listed():
    return [
        # One batch of a live stream: 32 spectra of four antennas, the filter history handed on from
        # batch to batch (file ingest at its smallest batches, where each call's latency counts).
        _fx("fx_chunk_4ant", 4, 4096, 32, 32, carry=True),
        # The plain correlator: 2^20 samples of four antennas into one dump.
        _fx("fx_plain_4ant", 4, 1024, 1024, 1024),
        # The headline: a 1 GiB real-time stream of four antennas, 16 dumps of 4096 spectra.
        _fx("fx_realtime_4ant", 4, 4096, 65536, 4096),
        # The large array at reduced precision: 32 antennas, spectra requantised to float16 and
        # correlated on the matrix cores.
        _fx("fx_32ant_f16", 32, 4096, 4096, 4096, x_prec="f16"),
        # An array of an odd size with the published filter (8-tap Kaiser, beta 8): two dumps and a
        # trailing partial one that is not integrated.
        _fx("fx_13ant_kaiser", 13, 2048, 1531, 700, n_taps=8, window="kaiser"),
        # Baseband I/Q words of 16 bits, as the acquisition chain delivers them.
        _fx("fx_iq16_4ant", 4, 4096, 16384, 4096, word="ci16"),
        # Five arrays of different sizes served together.
        {"name": "plan_5arrays", "kind": "plan", "arrays": "4:1024 8:2048 16:4096 24:4096 32:8192",
         "n_samp": 1 << 22, "mode": "graph"},
        # What follows each interval of the real-time stream: MAD flags, the delay and phase solve on
        # unflagged cells, and the current solution applied to the visibilities.
        {"name": "calibrate_4ant", "kind": "calibrate", "n_ant": 4, "n_time": 16, "n_chan": 2048},
        # Flags for an observation of 32 antennas: 528 baselines of 256 integrations x 2048 channels.
        {"name": "mad_plane_32ant", "kind": "mad", "n_time": 256, "n_base": 528, "n_chan": 2048,
         "population": 0, "sigma": 5.0},
        # The learned flagger over an 11-antenna observation (66 baselines), half activations.
        {"name": "flagger_66base_f16", "kind": "flagger", "n_time": 256, "n_base": 66, "n_chan": 2048,
         "act": "f16"},
        # One training step of the flagger on a batch of 32 tiles.
        {"name": "train_32tiles", "kind": "train", "n_img": 32, "height": 64, "width": 256},
        # An image of 32 antennas: 8.1 M visibilities onto 1024 x 1024, beam, 100 CLEAN components.
        {"name": "image_32ant_1024", "kind": "image", "n_ant": 32, "n_chan": 256, "n_time": 64, "n": 1024,
         "n_comp": 100},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["fx", "fx", "fx", "fx", "plan", "calibrate", "mad", "flagger", "train", "image"])
    if kind == "fx":
        word = rng.choice(["i8", "i8", "i8", "i16", "ci8", "ci16"])
        n_ant = rng.choice([2, 3, 4, 4, 4, 5, 8, 8, 13, 16, 24, 27, 32])
        n_fft = rng.choice([512, 1024, 2048, 4096, 4096, 8192])
        n_spec = max(9, _log_int(rng, 1 << 19, 1 << 27) // (n_ant * n_fft))
        per_dump = max(1, n_spec // rng.choice([1, 1, 2, 3, 7]))
        n_taps, window = rng.choice([(4, "hann"), (4, "hann"), (4, "hann"), (8, "kaiser"), (1, "rect")])
        x_prec = rng.choice(["f32", "f32", "f16", "bf16", "fp8"]) if n_ant > 4 else "f32"
        return _fx(None, n_ant, n_fft, n_spec, per_dump, n_taps=n_taps, window=window, word=word, x_prec=x_prec,
                   carry=n_taps > 1 and rng.random() < 0.4)
    if kind == "plan":
        arrays = ["%d:%d" % (rng.choice([2, 4, 8, 12, 16, 24, 32]), rng.choice([512, 1024, 2048, 4096, 8192]))
                  for _ in range(rng.randint(2, 5))]
        return {"kind": "plan", "arrays": " ".join(arrays), "n_samp": 8192 * _log_int(rng, 32, 512),
                "mode": rng.choice(["graph", "graph", "persistent"])}
    if kind == "calibrate":
        return {"kind": "calibrate", "n_ant": rng.randint(3, 32), "n_time": _log_int(rng, 4, 64),
                "n_chan": rng.choice([512, 1000, 1024, 2048, 4096])}
    if kind == "mad":
        n_time, n_chan = _log_int(rng, 8, 256), rng.choice([512, 1000, 2048, 4096])
        n_base = max(1, min(528, _log_int(rng, 1 << 18, 1 << 28) // (n_time * n_chan)))
        return {"kind": "mad", "n_time": n_time, "n_base": n_base, "n_chan": n_chan,
                "population": rng.choice([0, 0, 1, 2]), "sigma": rng.choice([3.0, 5.0])}
    if kind == "flagger":
        act = rng.choice(["f16", "f16", "f32"])
        n_time, n_chan = _log_int(rng, 16, 256), rng.choice([250, 512, 1024, 2048])
        most = (34 << 20) // (8 if act == "f32" else 1)
        n_base = max(1, min(66, _log_int(rng, 1 << 18, most) // (n_time * n_chan)))
        return {"kind": "flagger", "n_time": n_time, "n_base": n_base, "n_chan": n_chan, "act": act}
    if kind == "train":
        return {"kind": "train", "n_img": rng.randint(4, 32), "height": rng.choice([32, 50, 64]),
                "width": rng.choice([64, 100, 128, 256])}
    return {"kind": "image", "n_ant": rng.randint(4, 32), "n_chan": _log_int(rng, 16, 256),
            "n_time": _log_int(rng, 8, 64), "n": rng.choice([128, 256, 512, 1024]), "n_comp": rng.randint(10, 100)}


# ---- what a program has in hand before the call ------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device="cuda")


def _voltages(g, n_ant, n_samp, n_fft, word):
    """[n_ant, n_samp] (or [n_ant, n_samp, 2]) words: receiver noise, 30 % of the power common to all
    antennas at lags of 0..7 samples, and a line at one channel."""
    wide = word in ("i16", "ci16")
    sigma, top = (1200.0, 8191) if wide else (16.0, 127)
    parts = 2 if word in COMPLEX_WORDS else 1
    x = torch.empty((n_ant, n_samp, parts), dtype=torch.int16 if wide else torch.int8, device="cuda")
    k = n_fft // 7 + 1
    phase = 2 * math.pi * k / n_fft * torch.arange(n_fft, device="cuda", dtype=torch.float64)
    for q in range(parts):
        line = (sigma * 0.1 * torch.cos(phase - 0.5 * math.pi * q)).float()
        common = _randn(g, n_samp + 8)
        for a in range(n_ant):
            v = _randn(g, n_samp).mul_(sigma * math.sqrt(0.7))
            v += common[a % 8:a % 8 + n_samp] * (sigma * math.sqrt(0.3))
            v.view(-1, n_fft).add_(line)
            x[a, :, q] = v.round_().clamp_(-top, top)
    return x if parts == 2 else x.view(n_ant, n_samp)


def _n_samp(case):
    return case["n_spec"] * case["n_fft"]


def _params(g):
    """Network weights: He-scaled normal, small biases (flat: W1 b1 W2 b2 W3 b3 W4 b4)."""
    out = []
    for shape in ((32, 1, 3, 3), (32, 32, 5, 5), (32, 32, 5, 5), (1, 32, 1, 1)):
        fan_in = shape[1] * shape[2] * shape[3]
        out += [_randn(g, *shape).flatten() * math.sqrt(2.0 / fan_in), _randn(g, shape[0]) * 0.05]
    return torch.cat(out)


def _plane(g, n_time, n_base, n_chan):
    """Visibilities of an observation: complex noise, baselines at levels of their own, persistent lines
    and a few strong integrations."""
    level = 0.5 + _rand(g, 1, n_base, 1)
    vis = torch.empty((n_time, n_base, n_chan), dtype=torch.complex64, device="cuda")
    line = 1.0 + 9.0 * (_rand(g, n_chan) < 0.01)
    burst = 1.0 + 6.0 * (_rand(g, n_time, 1) < 0.03)
    ri = torch.view_as_real(vis)
    for t in range(n_time):
        ri[t] = _randn(g, n_base, n_chan, 2) * (level[0] * line * burst[t])[..., None]
    return vis


def _pairs(n_ant):
    return [(i, j) for i in range(n_ant) for j in range(i, n_ant)]


def _df(n_chan):
    return FS_HZ / (2 * n_chan)


def _solution(g, n_ant):
    tau = (_rand(g, n_ant) * 40e-9).double().cpu().tolist()
    phi = ((_rand(g, n_ant) - 0.5) * 2 * math.pi).double().cpu().tolist()
    return tau, phi


def _fringe(n_ant, n_chan, tau, phi):
    """exp(+i theta[b, k]) of the correction, complex128."""
    f = torch.arange(n_chan, device="cuda", dtype=torch.float64) * _df(n_chan)
    th = torch.stack([2 * math.pi * f * (tau[i] - tau[j]) + (phi[i] - phi[j]) for i, j in _pairs(n_ant)])
    return torch.polar(torch.ones_like(th), th)


def _uv(g, n_ant, n_chan, n_time):
    """(u, v) in wavelengths of all cross baselines, channels and hour angles: positions within 60 m,
    1.3-1.4 GHz, four hours at declination 58.8 degrees from latitude 36.7."""
    rad, ang = 60.0 * _rand(g, n_ant).double().sqrt(), 2 * math.pi * _rand(g, n_ant).double()
    east, north = rad * ang.cos(), rad * ang.sin()
    i, j = torch.triu_indices(n_ant, n_ant, 1, device="cuda")
    d_e, d_n = (east[j] - east[i])[:, None], (north[j] - north[i])[:, None]
    lat, dec = math.radians(36.7), math.radians(58.8)
    x, y, z = -math.sin(lat) * d_n, d_e, math.cos(lat) * d_n
    ha = torch.linspace(-30.0, 30.0, n_time, device="cuda", dtype=torch.float64) * (math.pi / 180)
    u = ha.sin() * x + ha.cos() * y
    v = -math.sin(dec) * ha.cos() * x + math.sin(dec) * ha.sin() * y + math.cos(dec) * z
    f = (1.30e9 + (torch.arange(n_chan, device="cuda", dtype=torch.float64) + 0.5) * (1.0e8 / n_chan)) / C_LIGHT
    return tuple((w[:, :, None] * f).float().flatten() for w in (u, v))


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "fx":
        n_ant, n_fft, n_taps = case["n_ant"], case["n_fft"], case["n_taps"]
        s = {"case": case, "x": _voltages(g, n_ant, _n_samp(case), n_fft, case["word"]), "taps": None,
             "hist": None, "hist_out": None}
        if case["window"] != "hann":
            s["taps"] = qc.design_taps(n_fft, n_taps, case["window"], 8.0)
        if case["carry"]:
            s["hist"] = _voltages(g, n_ant, (n_taps - 1) * n_fft, n_fft, case["word"])
            s["hist_out"] = torch.empty_like(s["hist"])
        return s
    if kind == "plan":
        arrays = _plan_arrays(case)
        plan = qc.Plan(arrays, mode=case["mode"])
        return {"case": case, "plan": plan, "vis": plan.empty_vis(),
                "x": [_voltages(g, a["n_ant"], a["n_samp"], a["n_fft"], "i8") for a in arrays]}
    if kind == "calibrate":
        n_ant, n_time, n_chan = case["n_ant"], case["n_time"], case["n_chan"]
        tau, phi = _solution(g, n_ant)
        vis = _randn(g, n_time, n_ant * (n_ant + 1) // 2, n_chan, 2)
        vis = torch.view_as_complex(vis) + 4.0 * _fringe(n_ant, n_chan, tau, phi).conj().to(torch.complex64)
        vis *= 1.0 + 29.0 * (_rand(g, n_chan) < 0.01)
        for b, (i, j) in enumerate(_pairs(n_ant)):
            if i == j:
                vis[:, b] = vis[:, b].abs() * 3.0
        return {"case": case, "vis": vis, "solution": _solution(g, n_ant)}
    if kind == "mad":
        return {"case": case, "vis": _plane(g, case["n_time"], case["n_base"], case["n_chan"])}
    if kind == "flagger":
        return {"case": case, "vis": _plane(g, case["n_time"], case["n_base"], case["n_chan"]), "params": _params(g)}
    if kind == "train":
        shape = (case["n_img"], case["height"], case["width"])
        labels = _rand(g, *shape) < 0.07
        r = _randn(g, *shape) * 1.2 + 6.0 * _rand(g, *shape) * labels
        params = _params(g)
        return {"case": case, "params": params, "x": torch.sign(r) * torch.log1p(r.abs()),
                "labels": labels.to(torch.uint8), "step": 200,
                "m": _randn(g, params.numel()) * 1e-3, "v": (_rand(g, params.numel()) * 1e-2 + 1e-3) ** 2}
    u, v = _uv(g, case["n_ant"], case["n_chan"], case["n_time"])
    cell = 1.0 / (4.0 * max(float(u.abs().max()), float(v.abs().max())))
    vis = _randn(g, u.numel(), 2)
    for flux, l, m in ((1.0, 0, 0), (0.5, 12, -7), (0.3, -20, 15)):
        ph = -2 * math.pi * torch.remainder((u.double() * l + v.double() * m) * cell, 1.0)
        vis[:, 0] += flux * ph.cos().float()
        vis[:, 1] += flux * ph.sin().float()
    return {"case": case, "u": u, "v": v, "vis": torch.view_as_complex(vis), "cell": cell}


def _plan_arrays(case):
    out = []
    for a in case["arrays"].split():
        n_ant, n_fft = (int(v) for v in a.split(":"))
        out.append({"n_ant": n_ant, "n_samp": case["n_samp"], "n_fft": n_fft, "n_taps": 4,
                    "spec_per_dump": case["n_samp"] // n_fft})
    return out


# ---- one pass ------------------------------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "fx":
        call = qc.xcorrelate if case["word"] == "i8" else qc.xcorrelate_ex
        vis = call(s["x"], case["n_fft"], case["n_taps"], case["per_dump"], taps=s["taps"], hist=s["hist"],
                   hist_out=s["hist_out"], x_prec=case["x_prec"])
        return {"vis": vis, "hist": s["hist_out"]}
    if kind == "plan":
        s["plan"].execute(s["x"], s["vis"])
        return s["vis"]
    if kind == "calibrate":
        n_ant, n_chan, vis = case["n_ant"], case["n_chan"], s["vis"]
        mask, thresh = qc.mad_flag(vis, 5.0, 0)
        done = qc.apply_delay_phase(vis.clone(), n_ant, 0.0, _df(n_chan), *s["solution"])
        tau, phi = qc.solve_delay_phase(vis, n_ant, 0.0, _df(n_chan), 0, n_chan // 8, n_chan - n_chan // 8, mask=mask)
        return {"mask": mask, "thresh": thresh, "vis": done, "tau": tau, "phi": phi}
    if kind == "mad":
        mask, thresh = qc.mad_flag(s["vis"], case["sigma"], case["population"])
        return {"mask": mask, "thresh": thresh}
    if kind == "flagger":
        return qc.cnn_forward(s["params"], qc.cnn_normalize(s["vis"]), act=case["act"])
    if kind == "train":
        loss = qc.cnn_train_step(s["params"], s["m"], s["v"], s["step"], s["x"], s["labels"], 13.0, lr=1e-3)
        s["step"] += 1
        return {"loss": loss, "params": s["params"], "m": s["m"], "v": s["v"]}
    dirty, psf = qc.image_dirty_and_psf(s["u"], s["v"], s["vis"], case["n"], s["cell"])
    residual = dirty.clone()
    pix, flux = qc.image_clean(residual, psf, 0.1, 1e-5, case["n_comp"])
    return {"dirty": dirty, "psf": psf, "pix": pix, "flux": flux, "residual": residual}


# ---- what a pass cannot do without ---------------------------------------------------------------

def _fx_work(n_ant, n_fft, n_taps, n_spec, n_dump, word="i8"):
    """Input and visibilities once; per input sample the filter (2P flop a component) and the transform,
    8 flop per baseline, channel and integrated spectrum."""
    cplx = word in COMPLEX_WORDS
    n_samp, n_chan = n_spec * n_fft, n_fft if cplx else n_fft // 2
    n_base = n_ant * (n_ant + 1) // 2
    per_samp = (2 * n_taps + 2.5 * math.log2(n_fft)) * (2 if cplx else 1)
    return (n_ant * n_samp * WORD_BYTES[word] + 8 * n_dump * n_base * n_chan,
            n_ant * n_samp * per_samp + 8 * n_base * n_chan * n_spec)


def work(case):
    kind = case["kind"]
    if kind == "fx":
        n_dump = case["n_spec"] // case["per_dump"]
        b, f = _fx_work(case["n_ant"], case["n_fft"], case["n_taps"], n_dump * case["per_dump"], n_dump, case["word"])
        if case["carry"]:
            b += 2 * case["n_ant"] * (case["n_taps"] - 1) * case["n_fft"] * WORD_BYTES[case["word"]]
        return {"bytes": b, "flops": f}
    if kind == "plan":
        each = [_fx_work(a["n_ant"], a["n_fft"], 4, a["spec_per_dump"], 1) for a in _plan_arrays(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    if kind == "calibrate":
        cells = case["n_time"] * case["n_ant"] * (case["n_ant"] + 1) // 2 * case["n_chan"]
        return {"bytes": 17 * cells, "flops": 24 * cells}
    if kind == "mad":
        cells = case["n_time"] * case["n_base"] * case["n_chan"]
        return {"bytes": 9 * cells, "flops": 6 * cells}
    if kind == "flagger":
        cells = case["n_time"] * case["n_base"] * case["n_chan"]
        return {"bytes": 12 * cells, "flops": 103104 * cells}
    if kind == "train":
        cells = case["n_img"] * case["height"] * case["width"]
        return {"bytes": 5 * cells, "flops": 3 * 103104 * cells}
    n_vis = case["n_ant"] * (case["n_ant"] - 1) // 2 * case["n_chan"] * case["n_time"]
    pixels = case["n"] * case["n"]
    return {"bytes": 16 * n_vis + 12 * pixels,
            "flops": 12 * n_vis + 10 * pixels * math.log2(pixels) + 2 * pixels * case["n_comp"]}


# ---- the same in 64 bits ---------------------------------------------------------------------------

def _taps64(n_fft, n_taps, window):
    if window == "rect":
        return torch.ones((n_taps, n_fft), device="cuda", dtype=torch.float64)
    size = n_fft * n_taps
    q = torch.arange(size, device="cuda", dtype=torch.float64)
    if window == "hann":
        w = 0.5 - 0.5 * torch.cos(2 * math.pi * q / (size - 1))
    else:
        r = 2 * q / (size - 1) - 1
        w = torch.special.i0(8.0 * torch.sqrt((1 - r * r).clamp_min(0))) / torch.special.i0(torch.full_like(q, 8.0))
    return (w * torch.sinc((q - (size - 1) / 2) / n_fft)).view(n_taps, n_fft)


def _fx64(x, hist, n_fft, n_taps, per_dump, window):
    """Visibilities complex128 of [n_ant, n_samp(, 2)] words."""
    n_ant, n_spec, cplx = x.shape[0], x.shape[1] // n_fft, x.dim() == 3
    taps = _taps64(n_fft, n_taps, window)
    if hist is None:
        hist = torch.zeros((n_ant, (n_taps - 1) * n_fft) + x.shape[2:], dtype=x.dtype, device=x.device)
    x = torch.cat((hist, x), 1)
    n_chan = n_fft if cplx else n_fft // 2
    i, j = torch.triu_indices(n_ant, n_ant, device="cuda")
    vis = torch.zeros((n_spec // per_dump, i.numel(), n_chan), dtype=torch.complex128, device="cuda")
    step = max(1, (1 << 25) // (n_ant * n_fft))
    for d in range(n_spec // per_dump):
        gram = torch.zeros((n_chan, n_ant, n_ant), dtype=torch.complex128, device="cuda")
        for m in range(d * per_dump, (d + 1) * per_dump, step):
            k = min(step, (d + 1) * per_dump - m)
            v = x[:, m * n_fft:(m + k + n_taps - 1) * n_fft].double()
            if cplx:
                v = torch.view_as_complex(v.contiguous())
            v = v.view(n_ant, k + n_taps - 1, n_fft)
            y = sum(v[:, p:p + k] * taps[p] for p in range(n_taps))
            f = torch.fft.fft(y) if cplx else torch.fft.rfft(y)[..., :n_chan]
            f = f.permute(2, 0, 1).contiguous()
            gram += torch.matmul(f, f.conj().transpose(1, 2).resolve_conj().contiguous())
        vis[d] = gram[:, i, j].t()
    return vis


def _median64(sorted_rows):
    k = sorted_rows.shape[-1]
    return 0.5 * (sorted_rows[..., (k - 1) // 2].double() + sorted_rows[..., k // 2].double())


def _mad64(amp):
    """(median, median absolute deviation), float64, over the last axis of float32 amplitudes."""
    med = _median64(amp.sort(-1).values)
    return med, _median64((amp.double() - med[..., None]).abs().sort(-1).values)


def _amplitudes(vis):
    return torch.view_as_real(vis).double().square().sum(-1).sqrt().float()


def _thresholds(vis, sigma, population):
    t, b, c = vis.shape
    out = []
    for k in range(b):
        amp = _amplitudes(vis[:, k])
        amp = amp.reshape(1, -1) if population == 0 else amp.t().contiguous() if population == 1 else amp
        med, mad = _mad64(amp)
        out.append(med + sigma * 1.4826 * mad)
    out = torch.stack(out)
    return out.view(b) if population == 0 else out if population == 1 else out.t().contiguous()


def _layers(params):
    out, at = [], 0
    for shape in ((32, 1, 3, 3), (32, 32, 5, 5), (32, 32, 5, 5), (1, 32, 1, 1)):
        size = shape[0] * shape[1] * shape[2] * shape[3]
        out.append((params[at:at + size].view(shape), params[at + size:at + size + shape[0]]))
        at += size + shape[0]
    return out


def _logits64(params, x):
    """[n, H, W] float64 logits; each convolution is a sum over its taps of 32 x 32 products."""
    n, height, width = x.shape
    a = x[None]
    for k, (w, bias) in enumerate(_layers(params)):
        dil = 2 if k == 2 else 1
        r = (w.shape[2] // 2) * dil
        pad = torch.nn.functional.pad(a, (r, r, r, r))
        z = bias[:, None]
        for ky in range(w.shape[2]):
            for kx in range(w.shape[3]):
                part = pad[:, :, ky * dil:ky * dil + height, kx * dil:kx * dil + width]
                z = z + w[:, :, ky, kx] @ part.reshape(part.shape[0], -1)
        a = (z.relu() if k < 3 else z).view(-1, n, height, width)
    return a[0]


def _clean64(dirty, psf, gain, n_comp):
    r, n = dirty.clone(), dirty.shape[0]
    flux = []
    for _ in range(n_comp):
        k = int(r.abs().argmax())
        g = gain * float(r.view(-1)[k])
        r -= g * torch.roll(psf, (k // n - n // 2, k % n - n // 2), (0, 1))
        flux.append(g)
    return torch.tensor(flux, dtype=torch.float64), r


def _dirty64(u, v, vis, n, cell):
    iu, iv = ((torch.floor(w.double() * (n * cell) + 0.5)).long() + n // 2 for w in (u, v))
    ok = (iu >= 0) & (iu < n) & (iv >= 0) & (iv < n) & (n - iu >= 0) & (n - iu < n) & (n - iv >= 0) & (n - iv < n)
    iu, iv, vis = iu[ok], iv[ok], torch.view_as_real(vis[ok].to(torch.complex128))
    grid = torch.zeros((n * n, 2), dtype=torch.float64, device="cuda")
    mirror = torch.tensor([1.0, -1.0], dtype=torch.float64, device="cuda")
    for part, at in ((vis, iu * n + iv), (vis * mirror, (n - iu) * n + (n - iv))):
        for q in range(2):
            grid[:, q] += torch.bincount(at, weights=part[:, q], minlength=n * n)
    grid = torch.view_as_complex(grid).view(n, n)
    image = torch.fft.fftshift(torch.fft.ifft2(torch.fft.ifftshift(grid))).real * (n * n)
    return image / (2.0 * iu.numel())


def exact(case, seed):
    s = prepare(case, seed)
    kind = case["kind"]
    if kind == "fx":
        return {"vis": _fx64(s["x"], s["hist"], case["n_fft"], case["n_taps"], case["per_dump"], case["window"]),
                "hist": None}
    if kind == "plan":
        return [_fx64(x, None, a["n_fft"], 4, a["spec_per_dump"], "hann")
                for x, a in zip(s["x"], _plan_arrays(case))]
    if kind == "calibrate":  # the solve's own values follow from float32 phases: no 64-bit value of the same steps
        vis = s["vis"].to(torch.complex128) * _fringe(case["n_ant"], case["n_chan"], *s["solution"])
        return {"mask": None, "thresh": _thresholds(s["vis"], 5.0, 0), "vis": vis, "tau": None, "phi": None}
    if kind == "mad":
        return {"mask": None, "thresh": _thresholds(s["vis"], case["sigma"], case["population"])}
    if kind == "flagger":
        params, out = s["params"].double(), []
        for b in range(case["n_base"]):
            amp = _amplitudes(s["vis"][:, b])
            med, mad = _mad64(amp.reshape(1, -1))
            scale = 1.4826 * float(mad) or 1.0
            r = (amp.double() - float(med)) / scale
            out.append(_logits64(params, (torch.sign(r) * torch.log1p(r.abs()))[None]))
        return torch.cat(out)
    if kind == "train":
        params = s["params"].double().requires_grad_(True)
        z, hot = _logits64(params, s["x"].double()), s["labels"] != 0
        soft = torch.nn.functional.softplus
        loss = torch.where(hot, 13.0 * soft(-z), soft(z)).mean()
        grad = torch.autograd.grad(loss, params)[0]
        m = 0.9 * s["m"].double() + 0.1 * grad
        v = 0.999 * s["v"].double() + 0.001 * grad * grad
        t = s["step"]
        new = params.detach() - 1e-3 * (m / (1 - 0.9 ** t)) / ((v / (1 - 0.999 ** t)).sqrt() + 1e-8)
        return {"loss": loss.detach().view(1), "params": new, "m": m, "v": v}
    dirty = _dirty64(s["u"], s["v"], s["vis"], case["n"], s["cell"])
    psf = _dirty64(s["u"], s["v"], torch.ones_like(s["vis"]), case["n"], s["cell"])
    flux, residual = _clean64(dirty, psf, 0.1, case["n_comp"])
    return {"dirty": dirty, "psf": psf, "pix": None, "flux": flux, "residual": residual}
