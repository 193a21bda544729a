"""Performance cases of the dedispersion library: what its users run.

Each case is one call (or one execute, or one serving round) through a public
entry point of ``paper_1509_00186_amd`` on resident data, with the buffers
that a program which calls it in a loop keeps:

beam        ``dedisperse`` of one channelised beam (optionally two
            polarisations, then ``fold`` at a pulse period)
plan        ``Plan.execute``: DM trials and/or several beams in one batch
fullband    ``fullband``: recorded spectra of a whole band, long real transforms
incoherent  ``incoherent``: the baseline without the coherent step
serving     ``Server``: blocks of a running stream pushed from host memory

Sizes are those of the repository's benchmark workloads and tests, and ragged
ones between them.  Inputs are Gaussian voltages as a recorder's 8-bit
quantiser (sigma 20) or a float pipeline (sigma 1) delivers them.
``exact`` evaluates the same definitions in 64 bits with plain torch.
"""
import math
import time

import numpy as np
import torch

import paper_1509_00186_amd as cdd

D_CONST = 4.148808e9  # us MHz^2 cm^3 / pc
TAPERS = ("none", "hann", "welch")


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def _beam(name, f, bw, nchan, nsamp, dm, fft_len=0, n_int=4, dtype="int8", taper="none",
          volt=False, chan=False, npol=1, bins=0, keep=True):
    c = dict(kind="beam", f=f, bw=bw, nchan=nchan, nsamp=nsamp, dm=dm, fft_len=fft_len,
             n_int=n_int, dtype=dtype, taper=taper, volt=volt, chan=chan, npol=npol, bins=bins,
             keep=keep)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # a first look at a short record: everything small, buffers not kept,
        # so launches and host work count
        _beam("beam_16ch_short", 325.0, 1.0, 16, 20_000, 67.9, 2048, volt=True, keep=False),
        # the 32 MHz GMRT beam, 4 s: the benchmark's own workload
        _beam("beam_512ch_4s", 325.0, 32.0, 512, 250_000, 67.9, 8192),
        # the upgraded 200 MHz band, 2 s
        _beam("beam_4096ch_2s", 400.0, 200.0, 4096, 97_656, 120.0, 8192),
        # a float pipeline's beam with odd channel count, length and
        # integration, tapered, length by the rule, every output wanted
        _beam("beam_ragged_cf32", 325.0, 6.3125, 101, 40_001, 26.8, 0, 3, "complex64", "hann",
              True, True),
        # two polarisations of a 1 s record, summed and folded at the pulse
        # period: the monitoring profile
        _beam("two_pol_fold_1s", 325.0, 32.0, 512, 62_500, 67.9, 8192, npol=2, bins=256),
        # one 16 MHz channel kept as baseband, long transforms, voltages out
        _beam("one_channel_2^23", 610.0, 16.0, 1, 1 << 23, 10.0, 1 << 18, 16, "complex64",
              volt=True),
        # a DM search: 64 evenly spaced trials on the 32 MHz beam
        dict(name="plan_64_trials", kind="plan", beams="325/32/512/250000/60:0.254:64",
             fft_len=2048, n_int=4, uneven=False),
        # four beams of uneven width and length in one plan, one DM each
        dict(name="plan_four_beams", kind="plan",
             beams="610/16/512/31250/10:0:1;325/32/512/125000/67.9:0:1;"
                   "325/32/1024/93750/67.9:0:1;400/200/4096/195312/120:0:1",
             fft_len=2048, n_int=4, uneven=False),
        # the unchannelised mode on half a second of 16 MHz records
        dict(name="fullband_2^24", kind="fullband", f=610.0, bw=16.0, nchan=512, nspec=16_384,
             dm=10.0, fft_len=0, n_int=16, taper="none", volt=False),
        # the same at the largest DM that fits its longest transform (4.2 s)
        dict(name="fullband_dm_limit", kind="fullband", f=610.0, bw=16.0, nchan=512,
             nspec=1 << 17, dm=3000.0, fft_len=0, n_int=16, taper="none", volt=False),
        # the quick look without coherent dedispersion
        dict(name="incoherent_512ch_4s", kind="incoherent", f=325.0, bw=32.0, nchan=512,
             nsamp=250_000, dm=67.9, n_int=4, dtype="int8", chan=False),
        # a live 32 MHz stream: blocks of 2^22 samples from host memory
        dict(name="serving_32MHz", kind="serving", f=325.0, bw=32.0, nchan=512, block=8192,
             blocks=6, dm=67.9, fft_len=0, n_int=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _band(rng, nchan):
    """A band of nchan channels like the recorded ones: (centre, width, DM)."""
    f, df = rng.choice([(325.0, 0.0625), (400.0, 200.0 / 4096), (610.0, 0.03125)])
    bw = min(nchan * df, 0.5 * f)
    # a DM whose sweep over the lowest channel stays below 500 samples
    lo, df = f - bw / 2, bw / nchan
    top = 500.0 / (D_CONST * df * (1 / lo ** 2 - 1 / (lo + df) ** 2))
    dm = math.exp(rng.uniform(math.log(5.0), math.log(min(300.0, top))))
    return f, bw, round(dm, 3)


def _length(rng, f, bw, nchan, dms, n_int, lo=256, hi=16384):
    n = _channel_plan(f, bw, nchan, dms, n_int, 0)[0]
    n = max(n, lo)
    return 1 << rng.randint(int(math.log2(n)), int(math.log2(hi)))


def draw(rng):
    kind = rng.choice(["beam"] * 5 + ["one"] * 2 + ["plan"] * 3 + ["fullband"] * 3 +
                      ["incoherent", "serving"])
    if kind == "beam":
        nchan = _log_int(rng, 4, 4096)
        nsamp = _log_int(rng, 4_000, min(400_000, 128_000_000 // nchan))
        f, bw, dm = _band(rng, nchan)
        n_int = rng.choice([1, 2, 3, 4, 4, 5, 8, 16])
        dtype = rng.choice(["int8", "int8", "int8", "complex64"])
        fft_len = rng.choice([0, _length(rng, f, bw, nchan, [dm], n_int)])
        volt = nchan * nsamp < 40_000_000 and rng.random() < 0.3
        npol = 2 if not volt and nchan * nsamp < 40_000_000 and rng.random() < 0.25 else 1
        return _beam("", f, bw, nchan, nsamp, dm, fft_len, n_int, dtype,
                     rng.choice(["none", "none", "hann", "welch"]), volt,
                     nchan * nsamp < 40_000_000 and rng.random() < 0.3, npol,
                     rng.choice([0, 64, 256, 1000]) if npol == 2 else 0, rng.random() < 0.7)
    if kind == "one":
        bw = rng.choice([16.0, 33.0])
        dm = round(math.exp(rng.uniform(math.log(1.0), math.log(30.0))), 3)
        nsamp = _log_int(rng, 1 << 20, 1 << 25)
        n = _channel_plan(610.0, bw, 1, [dm], 16, 0)[0]
        return _beam("", 610.0, bw, 1, nsamp, dm, rng.choice([0, 2 * n]),
                     rng.choice([3, 4, 16, 16]), rng.choice(["complex64", "complex64", "int8"]),
                     rng.choice(["none", "hann"]), rng.random() < 0.5)
    if kind == "plan":
        n_int = rng.choice([2, 4, 4, 5, 8])
        fft_len = rng.choice([1024, 2048, 2048, 4096, 8192])
        if rng.random() < 0.6:  # a DM search on one beam
            nchan = _log_int(rng, 8, 1024)
            ndm = _log_int(rng, 2, 64)
            nsamp = _log_int(rng, 4_000, max(4_001, min(250_000, 4_000_000_000 // (nchan * ndm))))
            f, bw, dm = _band(rng, nchan)
            beams = "%r/%r/%d/%d/%r:%r:%d" % (f, bw, nchan, nsamp, round(0.9 * dm, 3),
                                              round(0.1 * dm / ndm, 4), ndm)
        else:
            parts = []
            for _ in range(rng.randint(2, 4)):
                nchan = _log_int(rng, 8, 2048)
                nsamp = _log_int(rng, 4_000, 200_000)
                f, bw, dm = _band(rng, nchan)
                parts.append("%r/%r/%d/%d/%r:0:1" % (f, bw, nchan, nsamp, dm))
            beams = ";".join(parts)
        return dict(kind="plan", beams=beams, fft_len=fft_len, n_int=n_int,
                    uneven=rng.random() < 0.4)
    if kind == "fullband":
        nchan = rng.choice([128, 256, 512, 1024, 2048])
        bw = rng.choice([16.0, 33.0])
        # up to 2^27 real points by the length rule
        dm = round(math.exp(rng.uniform(math.log(1.0), math.log(1000.0 if bw < 20 else 600.0))), 3)
        nspec = _log_int(rng, (1 << 20) // (2 * nchan), (1 << 26) // (2 * nchan))
        return dict(kind="fullband", f=610.0, bw=bw, nchan=nchan, nspec=nspec, dm=dm, fft_len=0,
                    n_int=rng.choice([2, 6, 16, 16, 32]), taper=rng.choice(TAPERS),
                    volt=rng.random() < 0.3)
    if kind == "incoherent":
        nchan = _log_int(rng, 4, 4096)
        nsamp = _log_int(rng, 4_000, min(400_000, 128_000_000 // nchan))
        f, bw, dm = _band(rng, nchan)
        return dict(kind="incoherent", f=f, bw=bw, nchan=nchan, nsamp=nsamp, dm=dm,
                    n_int=rng.choice([1, 2, 3, 4, 8, 16]),
                    dtype=rng.choice(["int8", "int8", "complex64"]), chan=rng.random() < 0.3)
    nchan = rng.choice([256, 512, 1024])
    f, bw, dm = _band(rng, nchan)
    block, blocks = _log_int(rng, 2048, 8192), rng.randint(4, 8)
    # a sweep over the band of at most half of what a pass pushes
    sweep = 4.0 * int(_delays(f, bw, nchan, dm, 4).max())
    dm = round(dm * min(1.0, 0.5 * block * blocks / max(sweep, 1.0)), 3)
    return dict(kind="serving", f=f, bw=bw, nchan=nchan, block=block, blocks=blocks, dm=dm,
                fft_len=0, n_int=4)


# ---------------------------------------------------------------------------
# Inputs and passes
# ---------------------------------------------------------------------------
def _noise(shape, dtype, seed):
    """Seeded Gaussian voltages on the GPU, time-major."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    if dtype == "complex64":
        return torch.view_as_complex(torch.randn(*shape, 2, generator=g, device="cuda"))
    out = torch.empty(*shape, 2, dtype=torch.int8, device="cuda")
    flat = out.view(-1)
    step = 1 << 27
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        x = torch.randn(n, generator=g, device="cuda").mul_(20.0).round_().clamp_(-127, 127)
        flat[i:i + n] = x.to(torch.int8)
    return out


def _beams_of(case):
    """The beams of a plan case: dicts of f, bw, nchan, nsamp, dms."""
    out = []
    for part in case["beams"].split(";"):
        f, bw, nchan, nsamp, dm = part.split("/")
        d0, step, n = dm.split(":")
        d0, step, n = float(d0), float(step), int(n)
        dms = [d0 + step * i for i in range(n)]
        if case["uneven"]:
            dms = [d + 0.07 * step * (7 * i % 5) for i, d in enumerate(dms)]
        out.append(dict(f=float(f), bw=float(bw), nchan=int(nchan), nsamp=int(nsamp), dms=dms))
    return out


def _period(case):
    """Pulse period of 89 ms in integrated samples (at most a quarter of the series)."""
    t_int = case["nsamp"] // case["n_int"]
    return max(1.5, min(89e3 * case["bw"] / case["nchan"] / case["n_int"], t_int / 4.0))


def _input(case, seed):
    k = case["kind"]
    if k == "beam":
        shape = (case["nsamp"], case["nchan"])
        return _noise((2,) + shape if case["npol"] == 2 else shape, case["dtype"], seed)
    if k == "plan":
        return [_noise((b["nsamp"], b["nchan"]), "int8", 1000 * seed + i)
                for i, b in enumerate(_beams_of(case))]
    if k == "fullband":
        return _noise((case["nspec"], case["nchan"]), "int8", seed)
    if k == "incoherent":
        return _noise((case["nsamp"], case["nchan"]), case["dtype"], seed)
    return _noise((case["blocks"] * case["block"], case["nchan"]), "int8", seed).cpu().numpy()


def prepare(case, seed):
    x = _input(case, seed)
    s = dict(case=case, x=x, out=None)
    if case["kind"] == "plan":
        s["plan"] = cdd.Plan([dict(voltages=v, f_centre=b["f"], bw=b["bw"], dms=b["dms"],
                                   n_int=case["n_int"]) for v, b in zip(x, _beams_of(case))],
                             fft_len=case["fft_len"])
    elif case["kind"] == "serving":
        s["server"] = cdd.Server()
        s["sid"] = s["server"].open(cdd.CDD_CI8, case["nchan"], case["f"], case["bw"], case["dm"],
                                    case["n_int"], case["block"], case["fft_len"],
                                    block_len=case["block"])
        s["seq"] = 0
    elif case["kind"] == "fullband":
        i = cdd.fullband_query(case["nspec"], case["nchan"], case["f"], case["bw"], case["dm"],
                               case["n_int"], case["fft_len"], taper=case["taper"])
        s["out"] = dict(I=torch.empty(i["t_int"], device="cuda"),
                        ws=torch.empty(i["ws_bytes"], dtype=torch.uint8, device="cuda"))
        if case["volt"]:
            s["out"]["y"] = torch.empty(i["nsamp"], device="cuda")
    elif case["kind"] == "incoherent":
        t_int = case["nsamp"] // case["n_int"]
        dt = cdd.CDD_CI8 if case["dtype"] == "int8" else cdd.CDD_CF32
        n = cdd.lib.cdd_incoherent_ws_bytes(dt, case["nsamp"], case["nchan"], case["n_int"])
        s["out"] = dict(I=torch.empty(t_int, device="cuda"),
                        cov=torch.empty(t_int, dtype=torch.int32, device="cuda"),
                        ws=torch.empty(n, dtype=torch.uint8, device="cuda"))
        if case["chan"]:
            s["out"]["P"] = torch.empty(case["nchan"], t_int, device="cuda")
    elif case["keep"]:
        dt = cdd.CDD_CI8 if case["dtype"] == "int8" else cdd.CDD_CF32
        i = cdd.query(dt, case["nsamp"], case["nchan"], case["f"], case["bw"], case["dm"],
                      case["fft_len"], case["n_int"], case["volt"], taper=case["taper"])
        o = dict(I=torch.empty(i["t_int"], device="cuda"),
                 cov=torch.empty(i["t_int"], dtype=torch.int32, device="cuda"),
                 ws=torch.empty(i["ws_bytes"], dtype=torch.uint8, device="cuda"))
        if case["chan"]:
            o["P"] = torch.empty(case["nchan"], i["t_int"], device="cuda")
        if case["volt"]:
            o["y"] = torch.empty(case["nchan"], case["nsamp"], dtype=torch.complex64,
                                 device="cuda")
        s["out"] = o
    return s


def run(s):
    c, x = s["case"], s["x"]
    if c["kind"] == "beam":
        o = cdd.dedisperse(x, c["f"], c["bw"], c["dm"], c["fft_len"], c["n_int"],
                           want_chan=c["chan"], want_voltages=c["volt"], taper=c["taper"],
                           npol=c["npol"], out=s["out"])
        r = {k: o[k] for k in ("I", "cov", "P", "y") if k in o}
        if c["bins"]:
            r["profile"], r["counts"] = cdd.fold(o["I"], _period(c), 0.25, c["bins"])
        return r
    if c["kind"] == "plan":
        s["plan"].execute()
        return dict(I=s["plan"].I, cov=s["plan"].cov)
    if c["kind"] == "fullband":
        o = cdd.fullband(x, c["f"], c["bw"], c["dm"], c["n_int"], c["fft_len"], taper=c["taper"],
                         want_voltages=c["volt"], out=s["out"])
        return {k: o[k] for k in ("I", "y") if k in o}
    if c["kind"] == "incoherent":
        o = cdd.incoherent(x, c["f"], c["bw"], c["dm"], c["n_int"], want_chan=c["chan"],
                           out=s["out"])
        return {k: o[k] for k in ("I", "cov", "P") if k in o}
    sv, sid = s["server"], s["sid"]
    got = []
    for b in range(c["blocks"]):
        block = x[b * c["block"]:(b + 1) * c["block"]]
        while sv.push(sid, block, s["seq"]) != 0:  # queue full: collect results meanwhile
            got.append(sv.poll(sid)[1])
            time.sleep(0.0002)
        s["seq"] += 1
    sv.sync()
    got.append(sv.poll(sid)[1])
    return dict(I=np.concatenate(got))


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def _fft_flops(n):
    return 5.0 * n * math.log2(n)


def _beam_work(f, bw, nchan, nsamp, dms, fft_len, n_int):
    """Flops of one beam's transforms (the forward ones shared by its DMs),
    chirp products, detection and integration."""
    N, L, _ = _channel_plan(f, bw, nchan, dms, n_int, fft_len)
    blocks = nchan * -(-nsamp // (N - L))
    return blocks * (_fft_flops(N) + len(dms) * (_fft_flops(N) + 6.0 * N)) + \
        4.0 * nchan * nsamp * len(dms)


def work(case):
    k, n_int = case["kind"], case["n_int"]
    if k == "plan":
        by = fl = 0.0
        for b in _beams_of(case):
            by += 2.0 * b["nchan"] * b["nsamp"] + 8.0 * len(b["dms"]) * (b["nsamp"] // n_int)
            fl += _beam_work(b["f"], b["bw"], b["nchan"], b["nsamp"], b["dms"],
                             case["fft_len"], n_int)
        return dict(bytes=by, flops=fl)
    if k == "fullband":
        N, L, _ = _fullband_plan(case["f"] - case["bw"] / 2, case["bw"], case["dm"], n_int,
                                 case["fft_len"])
        T = case["nspec"] * 2 * case["nchan"]
        return dict(bytes=1.0 * T + 4.0 * (T // n_int) + (4.0 * T if case["volt"] else 0.0),
                    flops=0.5 * case["nspec"] * _fft_flops(2 * case["nchan"]) +
                    -(-T // (N - L)) * (_fft_flops(N) + 3.0 * N) + 2.0 * T)
    if k == "serving":
        T = case["blocks"] * case["block"]
        return dict(bytes=2.0 * case["nchan"] * T + 4.0 * (T // n_int),
                    flops=_beam_work(case["f"], case["bw"], case["nchan"], T, [case["dm"]],
                                     case["fft_len"], n_int))
    T, C = case["nsamp"], case["nchan"]
    es = 2 if case["dtype"] == "int8" else 8
    by = es * C * T + 8.0 * (T // n_int) + (4.0 * C * (T // n_int) if case["chan"] else 0.0)
    if k == "incoherent":
        return dict(bytes=by, flops=4.0 * C * T)
    fl = case["npol"] * _beam_work(case["f"], case["bw"], C, T, [case["dm"]], case["fft_len"],
                                   n_int)
    by += es * C * T * (case["npol"] - 1) + (8.0 * C * T if case["volt"] else 0.0)
    return dict(bytes=by + 8.0 * case["bins"], flops=fl + (T // n_int if case["bins"] else 0))


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------
def _pow2(x):
    p = 1
    while p < x:
        p *= 2
    return p


def _over(x):
    p = 1
    while not p > x:
        p *= 2
    return p


def _channel_plan(f, bw, nchan, dms, n_int, fft_len):
    """(N, L, nfront) of the channelised path."""
    df = bw / nchan
    fc = (f - bw / 2.0) + (np.arange(nchan) + 0.5) * df
    front = back = disp = 0.0
    for dm in dms:
        lo = D_CONST * dm * (1.0 / (fc * fc) - 1.0 / ((fc - df / 2) * (fc - df / 2))) * df
        hi = D_CONST * dm * (1.0 / (fc * fc) - 1.0 / ((fc + df / 2) * (fc + df / 2))) * df
        front = max(front, float(np.maximum(lo, hi).max()))
        back = max(back, float((-np.minimum(lo, hi)).max()))
        disp = max(disp, float((D_CONST * abs(dm) * (1.0 / (fc - df / 2) ** 2 -
                                                     1.0 / (fc + df / 2) ** 2) * df).max()))
    front, back = math.ceil(front), math.ceil(back)
    L = _pow2(max(1, front + back))
    N = fft_len or max(_over(2.0 * disp), 2 * L, 256)
    while L < N and (N - L) % n_int:
        L += 1
    nfront = front + (L - front - back) // 2
    if nfront - nfront % 16 >= front:
        nfront -= nfront % 16
    return N, L, nfront


def _fullband_plan(f_lo, bw, dm, n_int, fft_len):
    """(N, L, nfront) of the full-band path, real samples, dm >= 0."""
    reach = D_CONST * dm * (1.0 / (f_lo * f_lo) - 1.0 / ((f_lo + bw) * (f_lo + bw))) * (2.0 * bw)
    front = math.ceil(reach)
    L = _pow2(max(2, front))
    N = fft_len or max(_over(2.0 * reach), 2 * L, 1 << 16)
    while L < N and (N - L) % n_int:
        L += 1
    nf = front + (L - front) // 2
    if nf - nf % 32 >= front:
        nf -= nf % 32
    elif nf % 2:
        nf = nf + 1 if nf + 1 <= L else nf - 1
    return N, L, nf


def _window(x, taper):
    if taper == "hann":
        return 0.5 * (1.0 + torch.cos(2.0 * math.pi * x))
    return 1.0 - (2.0 * x) ** 2 if taper == "welch" else torch.ones_like(x)


def _turn(q):
    r = q - torch.round(q)
    return torch.polar(torch.ones_like(r), -2.0 * math.pi * r)


def _delays(f, bw, nchan, dm, n_int):
    df = bw / nchan
    fc = (f - bw / 2.0) + (np.arange(nchan) + 0.5) * df
    fref = fc[-1] if dm >= 0 else fc[0]
    return np.floor(D_CONST * dm * (1.0 / (fc * fc) - 1.0 / (fref * fref)) * df / n_int +
                    0.5).astype(np.int64)


def _integrate(p, n_int):
    t = p.shape[-1] // n_int
    return p[..., :t * n_int].reshape(p.shape[:-1] + (t, n_int)).sum(-1)


def _complex(v):
    """Time-major int8 or complex voltages -> complex128 [T][C]."""
    if v.dtype == torch.int8:
        v = torch.view_as_complex(v.double())
    return v.to(torch.complex128).reshape(v.shape[0], -1)


def _aligned(P, d, I, cov):
    """Add channel rows P [C][t_int], delayed by d, to I and cov."""
    t = I.shape[0]
    for p, k in zip(P, d.tolist()):
        if k < t:
            I[:t - k] += p[k:]
            cov[:t - k] += 1


def _coherent(v, f, bw, dms, n_int, fft_len, taper="none", each=None):
    """[(I, cov)] per DM; each(dm index, first channel, P, y) sees every group
    of channels."""
    T, C = v.shape[:2]
    N, L, nf = _channel_plan(f, bw, C, dms, n_int, fft_len)
    M, df, t_int = N - L, bw / C, T // n_int
    nblk = -(-T // M)
    dev = v.device
    res = [(torch.zeros(t_int, dtype=torch.float64, device=dev),
            torch.zeros(t_int, dtype=torch.int32, device=dev)) for _ in dms]
    s = torch.arange(N, dtype=torch.float64, device=dev)
    s = torch.where(s < N // 2, s, s - N)
    win = _window(s / N, taper)
    group = max(1, (1 << 26) // (nblk * N))
    for c0 in range(0, C, group):
        c1 = min(C, c0 + group)
        x = _complex(v[:, c0:c1]).T
        pad = torch.zeros(c1 - c0, (nblk - 1) * M + N, dtype=torch.complex128, device=dev)
        n = min(T, pad.shape[1] - nf)
        pad[:, nf:nf + n] = x[:, :n]
        X = torch.fft.fft(pad.unfold(1, N, M))
        del pad, x
        fc = (f - bw / 2.0) + (torch.arange(c0, c1, dtype=torch.float64, device=dev) + 0.5) * df
        off = s * df / N
        unit = D_CONST * off * off / ((fc * fc)[:, None] * (fc[:, None] + off))
        for i, dm in enumerate(dms):
            z = torch.fft.ifft(X * (_turn(unit * dm) * win)[:, None, :])
            y = z[:, :, nf:nf + M].reshape(c1 - c0, nblk * M)[:, :T]
            P = _integrate(y.real.square() + y.imag.square(), n_int)
            _aligned(P, _delays(f, bw, C, dm, n_int)[c0:c1], *res[i])
            if each is not None:
                each(i, c0, P, y)
            del z, y, P
    return res


def _exact_beam(case, x):
    C, T, n_int = case["nchan"], case["nsamp"], case["n_int"]
    t_int = T // n_int
    out = {}
    if case["chan"]:
        out["P"] = torch.zeros(C, t_int, dtype=torch.float64, device="cuda")
    if case["volt"]:
        out["y"] = torch.zeros(C, T, dtype=torch.complex128, device="cuda")

    def each(_, c0, P, y):
        if case["chan"]:
            out["P"][c0:c0 + len(P)] += P
        if case["volt"]:
            out["y"][c0:c0 + len(y)] = y

    for v in x if case["npol"] == 2 else [x]:
        (I, cov), = _coherent(v, case["f"], case["bw"], [case["dm"]], n_int, case["fft_len"],
                              case["taper"], each)
        out["I"], out["cov"] = out.get("I", 0) + I, cov
    if case["bins"]:
        u = np.arange(t_int, dtype=np.float64) / _period(case) + 0.25
        b = np.minimum(((u - np.floor(u)) * case["bins"]).astype(np.int64), case["bins"] - 1)
        out["profile"] = np.bincount(b, out["I"].cpu().numpy(), case["bins"])
        out["counts"] = np.bincount(b, minlength=case["bins"]).astype(np.int32)
    return out


def _exact_fullband(case, sp):
    nspec, C = sp.shape[:2]
    X = torch.zeros(nspec, C + 1, dtype=torch.complex128, device="cuda")
    X[:, :C] = _complex(sp)
    X[:, 0] = X[:, 0].real.clone().to(torch.complex128)
    x = torch.fft.irfft(X, n=2 * C).reshape(-1)
    del X
    f_lo, bw, n_int = case["f"] - case["bw"] / 2.0, case["bw"], case["n_int"]
    N, L, nf = _fullband_plan(f_lo, bw, case["dm"], n_int, case["fft_len"])
    M, T = N - L, x.shape[0]
    off = torch.arange(N // 2 + 1, dtype=torch.float64, device="cuda") * (bw / (N // 2))
    H = _turn(D_CONST * case["dm"] * off * off / (f_lo * f_lo * (f_lo + off)))
    H *= _window(off / bw - 0.5, case["taper"])
    del off
    y = torch.empty(T, dtype=torch.float64, device="cuda")
    group = max(1, (1 << 25) // N)
    nblk = -(-T // M)
    for k0 in range(0, nblk, group):
        k1 = min(nblk, k0 + group)
        seg = torch.zeros((k1 - k0 - 1) * M + N, dtype=torch.float64, device="cuda")
        a = k0 * M - nf
        lo, hi = max(0, a), min(T, a + seg.shape[0])
        seg[lo - a:hi - a] = x[lo:hi]
        Z = torch.fft.rfft(seg.unfold(0, N, M)) * H
        z = torch.fft.irfft(Z, n=N)[:, nf:nf + M].reshape(-1)
        n = min(T, k1 * M) - k0 * M
        y[k0 * M:k0 * M + n] = z[:n]
        del seg, Z, z
    out = dict(I=_integrate(y.square(), n_int))
    if case["volt"]:
        out["y"] = y
    return out


def exact(case, seed):
    x, k = _input(case, seed), case["kind"]
    if k == "beam":
        return _exact_beam(case, x)
    if k == "fullband":
        return _exact_fullband(case, x)
    if k == "plan":
        r = [_coherent(v, b["f"], b["bw"], b["dms"], case["n_int"], case["fft_len"])
             for v, b in zip(x, _beams_of(case))]
        return dict(I=[torch.stack([p[0] for p in b]) for b in r],
                    cov=[torch.stack([p[1] for p in b]) for b in r])
    if k == "incoherent":
        T, C, n_int = case["nsamp"], case["nchan"], case["n_int"]
        I = torch.zeros(T // n_int, dtype=torch.float64, device="cuda")
        cov = torch.zeros(T // n_int, dtype=torch.int32, device="cuda")
        d = _delays(case["f"], case["bw"], C, case["dm"], n_int)
        Ps = []
        for c0 in range(0, C, 64):
            v = _complex(x[:, c0:c0 + 64]).T
            P = _integrate(v.real.square() + v.imag.square(), n_int)
            _aligned(P, d[c0:c0 + 64], I, cov)
            if case["chan"]:
                Ps.append(P)
        return dict(I=I, cov=cov, **(dict(P=torch.cat(Ps)) if Ps else {}))
    # serving: the outputs that are final after a new stream's first blocks
    f, bw, C, n_int = case["f"], case["bw"], case["nchan"], case["n_int"]
    N, L, nf = _channel_plan(f, bw, C, [case["dm"]], n_int, case["fft_len"])
    (I, _), = _coherent(torch.from_numpy(x).cuda(), f, bw, [case["dm"]], n_int, case["fft_len"])
    done = max(0, (x.shape[0] + nf - N) // (N - L) + 1) * ((N - L) // n_int)
    n = max(0, done - int(_delays(f, bw, C, case["dm"], n_int).max()))
    return dict(I=I[:n].cpu().numpy())
