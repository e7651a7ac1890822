"""Performance cases of the lunar ns-pulse hot path.

Every case is work that a program of this library has it do through its
public entry points (paper_1612_06592_amd.lp): the whole chain on a block
(tiny, one beam, the 61-beam lunar tiling, the STEC search), single stages
at other shapes and types (int16 samples, wide bands, the 5 ns series),
two-stage beamforming, the station simulator, the PPF inversion and the
serving loop.  `draw` gives further cases of the same ranges.

Inputs are station noise with a few dispersed pulses, made on the GPU from
the seed.  Streams start past their start-up frames with the state an
earlier block would have left (the serving streams start fresh).

Not among the outputs: the offset of each frame's envelope maximum within
its frame.  Two samples of a frame whose envelopes agree within rounding
make it ambiguous even in 64 bits.  The offsets of the maxima that matter
come back in the trigger list's samples.
"""
import math
import random

import numpy as np
import torch

from paper_1612_06592_amd import lp

M, TAPS, NFFT, HOP, DELAY = 1024, 16, 4096, 2048, 1024
F0, FS, C_LIGHT = 100e6, 200e6, 299792458.0
_E, _EPS0, _ME = 1.602176634e-19, 8.8541878128e-12, 9.1093837015e-31
KAPPA = _E * _E / (8 * math.pi ** 2 * _EPS0 * _ME) * 1e16 / C_LIGHT
DEV = "cuda:0"


# ---------------------------------------------------------------- cases

def _chain(name, n_st, n_beams, k0, n_sb, n_t, dtype="ci8", prec="fp16",
           n_tec=1, tec0=10.0, tec1=10.0, group=0):
    return dict(name=name, kind="chain", n_st=n_st, n_beams=n_beams, k0=k0,
                n_sb=n_sb, n_t=n_t, dtype=dtype, prec=prec, n_tec=n_tec,
                tec0=tec0, tec1=tec1, group=group)


def listed():
    return [
        # The tiny workload: 4 stations, 32 subbands, 21 ms of data.  A call
        # of microseconds, where launches and latency count.
        _chain("chain-tiny", 4, 1, 189, 32, 4096, "ci16", tec0=5.0, tec1=5.0),
        # One beam at core scale: the ordinary block, 335 ms of data.
        _chain("chain-1beam", 24, 1, 52, 244, 65536),
        # The lunar tiling, 61 beams of 48 stations: the default bench
        # workload and the largest block of one STEC value.
        _chain("chain-61beams", 48, 61, 52, 244, 32768),
        # The slant TEC search: 7 beams at 32 trials, a quarter block.
        _chain("chain-search32", 24, 7, 52, 244, 16384, n_tec=32, tec0=0.0,
               tec1=30.0),
        # 16-bit samples (the rate the stations send) of all 48 stations:
        # rows too long for the matrix-core tile, so FP32 arithmetic.
        dict(name="beamform-ci16", kind="beamform", n_st=48, n_beams=37, k0=52,
             n_sb=122, n_t=8192, dtype="ci16", prec="fp32", gains=False),
        # Station gains and a ragged block: 36 stations, 19 beams, 39 rows of
        # 128 samples.
        dict(name="beamform-gains", kind="beamform", n_st=36, n_beams=19,
             k0=100, n_sb=311, n_t=4992, dtype="ci8", prec="fp16", gains=True),
        # De-dispersion of the widest served band, one serving chunk.
        dict(name="dedisperse-488", kind="dedisperse", n_beams=19, k0=24,
             n_sb=488, n_t=8192, n_tec=1, tec0=17.3, tec1=17.3),
        # The recovered 5 ns series itself, written out: 3 series.
        dict(name="synthesize-series", kind="synthesize", n_series=3, k0=60,
             n_sb=366, n_t=16384, series=True),
        # Stations too many for the link: preliminary beams of 8 groups, then
        # 61 final beams.
        dict(name="two-stage", kind="two_stage", n_st=48, n_groups=8,
             n_prelim=7, n_beams=61, k0=52, n_sb=122, n_t=8192),
        # The station simulator: noise, ADC and station filterbank.
        dict(name="station-sim", kind="station", n_in=48, k0=52, n_sb=244,
             n_frames=8177, words=16),
        # The exact PPF inversion of one beam, the paper's 25 iterations: a
        # pass applies the filterbank and its adjoint in turn.
        dict(name="lsmr-25", kind="lsmr", n_series=1, k0=52, n_sb=244,
             n_frames=32768, n_iter=25),
        # Blocks of four observation streams of uneven shapes through the
        # serving loop at once.
        dict(name="serve-4", kind="serve", streams=4, shapes=11,
             log2_lo=12, log2_hi=15),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["chain", "chain", "chain", "beamform", "dedisperse",
                       "synthesize", "two_stage", "station", "lsmr", "serve"])
    n_sb = _log(rng, 32, 488)
    k0 = rng.randint(1, 511 - n_sb)
    n_st = rng.randint(2, 24) * 2
    hops = _log(rng, 1, 32)
    beams = min(61, _log(rng, 1, 61))
    if kind == "chain":
        n_tec = rng.choice([1, 1, rng.randint(2, 32)])
        dtype = rng.choice(["ci8", "ci8", "ci16"])
        while (n_st * 2 * n_sb * hops * HOP > 7e8
               or beams * n_tec * n_sb * hops * HOP > 4e8
               or beams * n_tec * hops * HOP > 2e6):
            if hops > 1:
                hops -= 1
            elif beams > 1:
                beams -= 1
            else:
                n_tec -= 1
        t0 = rng.uniform(0.0, 15.0)
        c = _chain("", n_st, beams, k0, n_sb, hops * HOP, dtype,
                   "fp32" if dtype == "ci16" and n_st > 32 else "fp16", n_tec,
                   t0, t0 if n_tec == 1 else t0 + rng.uniform(1.0, 15.0),
                   rng.choice([0, rng.randint(1, n_tec)]) if n_tec > 1 else 0)
        del c["name"]
        return c
    if kind == "beamform":
        dtype = rng.choice(["ci8", "ci16"])
        prec = rng.choice(["fp16", "fp16", "fp32"])
        if dtype == "ci16" and n_st > 32:
            prec = "fp32"
        n_t = 128 * _log(rng, 1, 255)
        while n_st * 2 * n_sb * n_t > 4e8 or beams * n_sb * n_t > 2e8:
            n_t = 128 * (n_t // 256)
        return dict(kind=kind, n_st=n_st, n_beams=beams, k0=k0, n_sb=n_sb,
                    n_t=n_t, dtype=dtype, prec=prec,
                    gains=rng.choice([False, True]))
    if kind == "dedisperse":
        n_tec = rng.choice([1, rng.randint(2, 16)])
        while beams * n_tec * n_sb * hops * HOP > 2e8:
            if hops > 1:
                hops -= 1
            else:
                beams -= 1
        t0 = rng.uniform(0.0, 15.0)
        return dict(kind=kind, n_beams=beams, k0=k0, n_sb=n_sb,
                    n_t=hops * HOP, n_tec=n_tec, tec0=t0,
                    tec1=t0 if n_tec == 1 else t0 + rng.uniform(1.0, 15.0))
    if kind == "synthesize":
        series = rng.choice([False, True])
        n_series = _log(rng, 1, 61)
        while n_series * n_sb * hops * HOP > 2e8 or (
                n_series * hops * HOP > (2e5 if series else 1e6)):
            if hops > 1:
                hops -= 1
            else:
                n_series -= 1
        return dict(kind=kind, n_series=n_series, k0=k0, n_sb=n_sb,
                    n_t=hops * HOP, series=series)
    if kind == "two_stage":
        g, p = rng.choice([(4, 7), (6, 7), (8, 7), (12, 5), (10, 1)])
        n_st = max(n_st, g)
        n_t = 128 * _log(rng, 1, 80)
        while n_st * 2 * n_sb * n_t > 2e8 or 61 * n_sb * n_t > 2e8:
            n_t = 128 * (n_t // 256)
        return dict(kind=kind, n_st=n_st, n_groups=g, n_prelim=p,
                    n_beams=beams, k0=k0, n_sb=n_sb, n_t=n_t)
    if kind == "station":
        n_in = rng.randint(1, 96)
        return dict(kind=kind, n_in=n_in, k0=k0, n_sb=n_sb,
                    n_frames=_log(rng, 64, 390000 // n_in),
                    words=rng.randint(1, 24))
    if kind == "lsmr":
        n_series = rng.randint(1, 4)
        return dict(kind=kind, n_series=n_series, k0=k0, n_sb=n_sb,
                    n_frames=_log(rng, 64, 32000 // n_series),
                    n_iter=rng.randint(5, 25))
    return dict(kind="serve", streams=rng.randint(2, 5),
                shapes=rng.randint(0, 10 ** 6), log2_lo=11, log2_hi=14)


def _streams(case):
    """Shapes of the serving case's streams."""
    r = random.Random(case["shapes"])
    out = []
    for _ in range(case["streams"]):
        n_sb = 122 * r.randint(1, 4)
        out.append(dict(n_st=4 * r.randint(6, 12),
                        n_beams=r.choice([7, 19, 37, 61]),
                        k0=min(52, 512 - n_sb), n_sb=n_sb,
                        tec0=r.uniform(0.0, 30.0),
                        n_t=2 ** r.randint(case["log2_lo"], case["log2_hi"])))
    return out


# --------------------------------------------------------------- inputs

def _tec(case):
    t0 = case.get("tec0", 10.0)
    return np.linspace(t0, case.get("tec1", t0), case.get("n_tec", 1))


def _k(case):
    return np.arange(case["k0"], case["k0"] + case["n_sb"], dtype=np.int32)


def _freq(k):
    return F0 + np.asarray(k, dtype=np.float64) * FS / M


def _unit(azel):
    az, el = azel[:, 0], azel[:, 1]
    return np.stack([np.cos(el) * np.sin(az), np.cos(el) * np.cos(az),
                     np.sin(el)], 1)


def _geometry(rng, n_st, n_beams):
    """Stations in a 2 km disk and beams tiling the Moon at 0.1 deg."""
    r = 1000.0 * np.sqrt(rng.uniform(0, 1, n_st))
    phi = rng.uniform(0, 2 * np.pi, n_st)
    enu = np.stack([r * np.sin(phi), r * np.cos(phi), np.zeros(n_st)], 1)
    az0, el0 = rng.uniform(0, 2 * np.pi), np.deg2rad(rng.uniform(25, 65))
    q = np.array([(i, j) for i in range(-5, 6) for j in range(-5, 6)])
    uv = np.stack([q[:, 0] + 0.5 * q[:, 1], np.sqrt(0.75) * q[:, 1]], 1)
    uv = uv[np.argsort((uv ** 2).sum(1), kind="stable")][:n_beams]
    uv = np.deg2rad(0.1) * uv
    return enu, np.stack([az0 + uv[:, 0] / np.cos(el0), el0 + uv[:, 1]], 1)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _voltages(rng, gen, case, enu, azel, n_pulses=3):
    """Station subbands [S][T][n_in][2]: noise with dispersed pulses that
    come from beam directions at random frames."""
    S, T, n_in = case["n_sb"], case["n_t"], 2 * case["n_st"]
    wide = case.get("dtype", "ci8") == "ci16"
    sigma, lim = (16.0, 32767) if wide else (8.0, 127)
    x = torch.empty((S, T, n_in, 2), dtype=torch.int16 if wide else torch.int8,
                    device=DEV)
    f = _freq(_k(case))
    tec = _tec(case)
    pulses = []
    for _ in range(n_pulses):
        n = _unit(azel[rng.integers(len(azel))][None])[0]
        ph = (f[:, None] * (enu @ n)[None] / C_LIGHT
              + (KAPPA * tec[len(tec) // 2] / f)[:, None]
              - (_k(case) * rng.integers(M) / M)[:, None])
        a = sigma * rng.uniform(8, 15) / math.sqrt(S * n_in)
        z = np.repeat(a * np.exp(2j * np.pi * ph), 2, axis=1)
        pulses.append((int(rng.integers(T)), torch.from_numpy(
            np.stack([z.real, z.imag], -1).astype(np.float32)).to(DEV)))
    step = max(1, (1 << 26) // (T * n_in * 2))
    for s in range(0, S, step):
        e = min(S, s + step)
        v = torch.randn((e - s, T, n_in, 2), generator=gen, device=DEV)
        v *= sigma
        for m, z in pulses:
            v[:, m] += z[s:e]
        x[s:e] = v.round_().clamp_(-lim, lim).to(x.dtype)
    return x


def _fill(gen, buf, rms):
    """A cf32 state or data buffer filled with noise of this rms per part."""
    v = buf.view(torch.float32)
    step = 1 << 28
    for i in range(0, v.numel(), step):
        v[i:i + step].normal_(0.0, rms, generator=gen)


def _dtype(case):
    return lp.LP_CI16 if case.get("dtype") == "ci16" else lp.LP_CI8


def _prec(case):
    return lp.LP_FP32 if case.get("prec") == "fp32" else lp.LP_FP16_MFMA


def _zeros(*shape):
    return torch.zeros(shape, dtype=torch.float32, device=DEV)


def _empty(*shape):
    return torch.empty(shape, dtype=torch.float32, device=DEV)


def _gains(rng, case):
    n = 2 * case["n_st"]
    return rng.uniform(0.3, 3.0, n).astype(np.float32) if case["gains"] else None


class _Served:
    """A server with its open streams; the server goes before its context."""

    def __init__(self, case, seed):
        rng, gen = np.random.default_rng(seed), _gen(seed)
        self.ctx = lp.Ctx(0)
        self.shapes = _streams(case)
        self.geom, self.blocks, cfgs, need = [], [], [], 0
        for c in self.shapes:
            enu, azel = _geometry(rng, c["n_st"], c["n_beams"])
            self.geom.append((enu, azel))
            self.blocks.append(_voltages(rng, gen, c, enu, azel))
            cfg = lp.StreamCfg(enu, _k(c), azel, _tec(c), c["n_t"])
            need += cfg.resident_bytes() + 2 * cfg.block_bytes(c["n_t"])
            cfgs.append(cfg)
        torch.cuda.synchronize()
        self.arena = torch.empty(need + (64 << 20), dtype=torch.uint8,
                                 device=DEV)
        self.srv = lp.Server(self.ctx, self.arena)
        self.ids = [self.srv.open(cfg) for cfg in cfgs]

    def __del__(self):
        if hasattr(self, "srv"):
            self.srv.destroy()
        self.ctx.close()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        return dict(kind=kind, served=_Served(case, seed))
    rng, gen = np.random.default_rng(seed), _gen(seed)
    ctx = lp.Ctx(0)
    band = lp.Band(_k(case))
    st = dict(kind=kind, ctx=ctx, band=band, case=case)
    S, n_t = case["n_sb"], case.get("n_t", 0)
    if kind == "chain":
        enu, azel = _geometry(rng, case["n_st"], case["n_beams"])
        p = lp.Pipeline(ctx, lp.Array(enu, 2), band, lp.Dirs(azel), _tec(case),
                        n_t, dtype=_dtype(case), prec=_prec(case),
                        trial_group=case["group"])
        p.frame0 = 8 * n_t
        rms = (16.0 if case["dtype"] == "ci16" else 8.0) * math.sqrt(
            2 * case["n_st"])
        _fill(gen, p.bufs["tail"], rms)
        _fill(gen, p.bufs["hist"], rms)
        st.update(p=p, x=_voltages(rng, gen, case, enu, azel), enu=enu,
                  azel=azel)
        trig = p.bufs["trig"].view(torch.int32).view(-1, 6)
        emax, _, psum = p.cand_view()
        B, J = case["n_beams"], case["n_tec"]
        out = dict(y=p.y_view(), emax=emax, psum=psum, sigma=p.bufs["sigma"],
                   snr=p.bufs["snr"], best=p.bufs["best"],
                   n_trig=p.bufs["n_trig"], trig=trig[:, :4],
                   trig_snr=trig[:, 4:].view(torch.float32),
                   tail=p.bufs["tail"].view(torch.float32).view(B, S, -1, 2),
                   hist=p.bufs["hist"].view(torch.float32).view(B * J, S, 16, 2))
        if not case["group"]:
            out["d"] = p.d_view()
        st["out"] = out
    elif kind == "beamform":
        enu, azel = _geometry(rng, case["n_st"], case["n_beams"])
        gain = _gains(rng, case)
        st.update(enu=enu, azel=azel, gain=gain,
                  array=lp.Array(enu, 2, gain), dirs=lp.Dirs(azel),
                  x=_voltages(rng, gen, case, enu, azel),
                  y=_empty(case["n_beams"], S, n_t, 2))
    elif kind == "dedisperse":
        B, J = case["n_beams"], case["n_tec"]
        st.update(tec=_tec(case), y=_empty(B, S, n_t, 2),
                  tail=_zeros(B, S, HOP, 2), d=_empty(B, J, S, n_t, 2))
        _fill(gen, st["y"], 60.0)
        _fill(gen, st["tail"], 60.0)
    elif kind == "synthesize":
        ns = case["n_series"]
        st.update(d=_empty(ns, S, n_t, 2), hist=_zeros(ns, S, 16, 2),
                  cand=torch.empty(lp.nbytes("lp_cand_bytes", ns, n_t),
                                   dtype=torch.uint8, device=DEV),
                  x_out=_empty(ns, n_t * M) if case["series"] else None)
        _fill(gen, st["d"], 60.0)
        _fill(gen, st["hist"], 60.0)
        head = st["cand"][:ns * n_t * 8].view(torch.float32).view(ns, n_t, 2)
        out = dict(emax=head[..., 0], hist=st["hist"],
                   psum=st["cand"][ns * n_t * 8:][:ns * n_t // 4].view(
                       torch.float32).view(ns, n_t // 16))
        if case["series"]:
            out["series"] = st["x_out"]
        st["out"] = out
    elif kind == "two_stage":
        enu, azel = _geometry(rng, case["n_st"], case["n_beams"])
        _, prelim = _geometry(rng, 1, case["n_prelim"])
        # Wider apart than the final beams, and off their lattice so that no
        # final beam is as near to one preliminary beam as to another.
        prelim = 2.6 * (prelim - prelim[0]) + azel[0] + [1.1e-4, 2.3e-4]
        G = case["n_groups"]
        group = np.argsort(np.argsort(np.arctan2(enu[:, 0], enu[:, 1]))) \
            * G // case["n_st"]
        st.update(enu=enu, azel=azel, prelim_azel=prelim, group=group,
                  array=lp.Array(enu, 2), dirs=lp.Dirs(azel),
                  prelim=lp.Dirs(prelim), groups=lp.Groups(group, G),
                  x=_voltages(rng, gen, case, enu, azel),
                  y1=_empty(G * case["n_prelim"], S, n_t, 2),
                  y=_empty(case["n_beams"], S, n_t, 2))
    elif kind == "station":
        n_in, nf = case["n_in"], case["n_frames"]
        st.update(seed=int(seed), pulse=torch.randn(
                      (n_in, 4000), generator=gen, device=DEV) * 40.0,
                  adc=torch.empty((n_in, (nf + 15) * M), dtype=torch.int16,
                                  device=DEV),
                  x=torch.empty((S, nf, n_in, 2), dtype=torch.int8, device=DEV),
                  work=torch.empty(lp.nbytes("lp_station_work_bytes", n_in, S,
                                             nf), dtype=torch.uint8,
                                   device=DEV))
    elif kind == "lsmr":
        ns, nf = case["n_series"], case["n_frames"]
        st.update(y=_empty(ns, S, nf, 2), x=_empty(ns, (nf - 15) * M),
                  work=torch.empty(lp.nbytes("lp_ppf_work_bytes", S, ns, nf),
                                   dtype=torch.uint8, device=DEV))
        _fill(gen, st["y"], 60.0)
    return st


def run(st):
    kind, case = st["kind"], st.get("case")
    if kind == "chain":
        st["p"].step(st["x"])
        return st["out"]
    if kind == "serve":
        s = st["served"]
        for i, (sid, x, c) in enumerate(zip(s.ids, s.blocks, s.shapes)):
            s.srv.submit(sid, x, c["n_t"], tag=i)
        got = []
        while len(got) < len(s.ids):
            got += s.srv.poll()
        got.sort(key=lambda r: r["tag"])
        out = []
        for r in got:
            t = np.zeros(1024, lp.TRIG_DTYPE)   # the streams' trigger limit
            t[:len(r["trig"])] = r["trig"]
            out.append(dict(n_trig=r["n_trig"], snr=r["snr"],
                            best=r["best_tec"], sample=t["sample"],
                            beam=t["beam"], tec=t["tec"], trig_snr=t["snr"]))
        return out
    ctx, band = st["ctx"], st["band"]
    if kind == "beamform":
        lp.beamform(ctx, st["array"], band, st["dirs"], st["x"], case["n_t"],
                    _dtype(case), _prec(case), st["y"])
        return st["y"]
    if kind == "dedisperse":
        lp.dedisperse(ctx, band, st["tec"], st["y"], case["n_beams"],
                      case["n_t"], st["tail"], st["d"])
        return dict(d=st["d"], tail=st["tail"])
    if kind == "synthesize":
        lp.synthesize(ctx, band, st["d"], case["n_series"], case["n_t"],
                      8 * case["n_t"], st["hist"], st["cand"], st["x_out"])
        return st["out"]
    if kind == "two_stage":
        lp.beamform_groups(ctx, st["array"], st["groups"], band, st["prelim"],
                           st["x"], case["n_t"], st["y1"])
        lp.beamform_stage2(ctx, st["array"], st["groups"], band, st["prelim"],
                           st["dirs"], st["y1"], case["n_t"], st["y"])
        return dict(y1=st["y1"], y=st["y"])
    if kind == "station":
        n_in, nf = case["n_in"], case["n_frames"]
        lp.sim_adc(ctx, st["seed"], n_in, case["words"], 12, 0,
                   (nf + 15) * M, st["adc"], st["pulse"], 20 * M + 77)
        lp.station_ppf(ctx, band, st["adc"], n_in, nf, 0.6, st["x"],
                       st["work"])
        return dict(adc=st["adc"], x=st["x"])
    lp.ppf_invert(ctx, band, st["y"], case["n_series"], case["n_frames"],
                  case["n_iter"], st["x"], st["work"])
    return st["x"]


# ----------------------------------------------------------------- work

def work(case):
    kind, S = case["kind"], case.get("n_sb", 0)
    n_t, B = case.get("n_t", 0), case.get("n_beams", 1)
    if kind == "serve":
        # group: the beams and de-dispersed subbands stay in the server.
        w = [_work_chain(dict(c, dtype="ci8", n_tec=1, group=1))
             for c in _streams(case)]
        return {q: sum(v[q] for v in w) for q in ("bytes", "flops")}
    if kind == "chain":
        return _work_chain(case)
    if kind in ("beamform", "two_stage"):
        n_in = 2 * case["n_st"]
        xb = S * n_t * n_in * (4 if case.get("dtype") == "ci16" else 2)
        if kind == "beamform":
            return dict(bytes=xb + 8 * B * S * n_t,
                        flops=8 * n_in * B * S * n_t)
        G, P = case["n_groups"], case["n_prelim"]
        return dict(bytes=xb + 8 * S * n_t * (G * P + B),
                    flops=8 * S * n_t * (n_in * P + G * B))
    if kind == "dedisperse":
        J = case["n_tec"]
        return dict(bytes=8 * B * S * (n_t * (1 + J) + 2 * HOP),
                    flops=B * S * n_t * (120 + 132 * J))
    if kind == "synthesize":
        ns = case["n_series"]
        return dict(bytes=8 * ns * S * (n_t + 32) + ns * n_t * 8.25
                    + (4 * ns * n_t * M if case["series"] else 0),
                    flops=120 * ns * n_t * M)
    if kind == "station":
        n_in, nf = case["n_in"], case["n_frames"]
        n = n_in * (nf + 15) * M
        # 80 products and as many three-input xors per group of four words.
        return dict(bytes=2 * n + 2 * n_in * S * nf,
                    flops=n * (160 * ((case["words"] + 3) // 4) + 60))
    ns, nf, it = case["n_series"], case["n_frames"], case["n_iter"]
    # An iteration cannot do without u read and written, v read and written
    # and x; the vectors of one solve do not fit in any cache.
    return dict(bytes=ns * ((it + 1) * (16 * S * nf + 8 * M * (nf - 15))
                            + 4 * M * (nf - 15)),
                flops=ns * (2 * it + 1) * 57 * M * nf)


def _work_chain(c):
    S, n_t, B, J = c["n_sb"], c["n_t"], c["n_beams"], c["n_tec"]
    n_in = 2 * c["n_st"]
    b = S * n_t * n_in * (4 if c["dtype"] == "ci16" else 2)
    b += B * J * n_t * 8 + 16 * S * (B * HOP + 16 * B * J)
    if not c["group"]:  # the beams and the de-dispersed subbands are kept
        b += 8 * B * S * n_t * (1 + J)
    return dict(bytes=b, flops=S * n_t * B * (8 * n_in + 120 + 132 * J)
                + 120 * B * J * n_t * M)


# ------------------------------------------------- the same in 64 bits

def _as_c128(t):
    return torch.view_as_complex(t.double().contiguous())


def _real(z):
    return torch.view_as_real(z)


def _weights(enu, azel, k, gain=None, n_pol=2):
    """[S][B][n_in] complex: gain exp(-2 pi i f (r . n) / c)."""
    cyc = _freq(k)[:, None, None] * (_unit(azel) @ enu.T)[None] / C_LIGHT
    w = np.repeat(np.exp(-2j * np.pi * (cyc - np.floor(cyc))), n_pol, axis=2)
    if gain is not None:
        w = w * np.asarray(gain, dtype=np.float64)[None, None]
    return torch.from_numpy(w).to(DEV)


def _exact_beams(x, w):
    """[B][S][T] complex from [S][T][n_in][2] and [S][B][n_in]."""
    S, T = x.shape[:2]
    y = torch.empty((w.shape[1], S, T), dtype=torch.complex128, device=DEV)
    for s in range(S):
        y[:, s] = (_as_c128(x[s]) @ w[s].T.contiguous()).T
    return y


def _chirp(k, tec):
    q = torch.arange(NFFT, device=DEV, dtype=torch.float64)
    q = torch.where(q >= NFFT // 2, q - NFFT, q)
    f = torch.from_numpy(_freq(k)).to(DEV)[:, None]
    c = KAPPA * float(tec) / (f + q * (FS / M / NFFT)) + q * (DELAY / NFFT)
    c = -2 * math.pi * (c - torch.floor(c))
    return torch.complex(torch.cos(c), torch.sin(c))


def _exact_dedisperse(y, tail, k, tec):
    """[S][T] complex of one beam at one trial, with its [S][2048] tail."""
    v = torch.cat([tail, y], 1).unfold(1, NFFT, HOP)       # [S][hops][4096]
    v = torch.fft.ifft(torch.fft.fft(v) * _chirp(k, tec)[:, None])
    return v[..., NFFT - HOP:].reshape(y.shape)


def _prototype():
    n = M * TAPS
    h = np.kaiser(n, 9.0) * np.sinc((np.arange(n) - 0.5 * (n - 1)) / M)
    return torch.from_numpy((h / h.sum()).reshape(TAPS, M)).to(DEV)


def _exact_series(d, hist, k, want=False):
    """(emax, psum, series or None) of one series [S][T], history [S][16]."""
    g = M * _prototype()
    T = d.shape[1]
    d = torch.cat([hist, d], 1)
    emax = torch.empty(T, dtype=torch.float64, device=DEV)
    psum = torch.empty(T // 16, dtype=torch.float64, device=DEV)
    series = torch.empty(T * M, dtype=torch.float64, device=DEV) if want else None
    kk = torch.from_numpy(k.astype(np.int64)).to(DEV)
    step = 4096
    for m in range(0, T, step):
        e = min(T, m + step)
        z = torch.zeros((e - m + 16, M), dtype=torch.complex128, device=DEV)
        z[:, kk] = d[:, m:e + 16].T
        z = torch.fft.ifft(z) * M
        o = torch.zeros((e - m, M), dtype=torch.complex128, device=DEV)
        for t in range(TAPS):
            o += g[t] * z[16 - t:16 - t + e - m]
        emax[m:e] = 2 * o.abs().amax(1)
        re = 2 * o.real
        psum[m // 16:e // 16] = (re * re).view((e - m) // 16, -1).sum(1)
        if want:
            series[m * M:e * M] = re.reshape(-1)
    return emax, psum, series


def _exact_chain(case, x, enu, azel, tail, hist, first=0, keep=True):
    """The chain's outputs on one block in 64 bits; frames before `first` are
    not in the statistics."""
    k, tec = _k(case), _tec(case)
    y = _exact_beams(x, _weights(enu, azel, k))
    B, S, T = y.shape
    J = len(tec)
    d = torch.empty((B, J, S, T), dtype=torch.complex128, device=DEV) \
        if keep else None
    emax = torch.empty((B * J, T), dtype=torch.float64, device=DEV)
    psum = torch.empty((B * J, T // 16), dtype=torch.float64, device=DEV)
    power = torch.empty(B * J, dtype=torch.float64, device=DEV)
    h2 = torch.empty((B * J, S, 16), dtype=torch.complex128, device=DEV)
    for b in range(B):
        for j in range(J):
            i = b * J + j
            v = _exact_dedisperse(y[b], tail[b], k, tec[j])
            if keep:
                d[b, j] = v
            h2[i] = v[:, -16:]
            emax[i], psum[i], _ = _exact_series(v, hist[i], k)
            power[i] = psum[i, first // 16:].sum()
    sigma = torch.sqrt(power / ((T - first) * M))
    snr = emax[:, first:].amax(1) / sigma
    return dict(y=_real(y), d=_real(d) if keep else None, emax=emax, psum=psum,
                sigma=sigma.view(B, J), snr=snr.view(B, J),
                tail=_real(y[:, :, T - HOP:]), hist=_real(h2), best=None,
                n_trig=None, trig=None, trig_snr=None)


def _analysis(h, k, x):
    """H x: [S][n_frames] complex of a real series of F frames."""
    xr = x.view(-1, M).flip(1)
    v = torch.zeros((xr.shape[0] + TAPS - 1, M), dtype=torch.float64,
                    device=DEV)
    for t in range(TAPS):
        v[t:t + xr.shape[0]] += h[t] * xr
    return torch.fft.rfft(v)[:, k].conj().T.contiguous()


def _adjoint(h, k, y):
    """H^T y, the real adjoint."""
    s = torch.zeros((y.shape[1], M // 2 + 1), dtype=torch.complex128,
                    device=DEV)
    s[:, k] = y.conj().T
    w = torch.fft.irfft(s, n=M) * (M / 2)
    F = y.shape[1] - TAPS + 1
    xr = torch.zeros((F, M), dtype=torch.float64, device=DEV)
    for t in range(TAPS):
        xr += h[t] * w[t:t + F]
    return xr.flip(1).reshape(-1)


def _lsmr(h, k, b, n_iter):
    """LSMR (Fong & Saunders 2011, Algorithm 1) from 0, no damping."""
    def norm(a):
        return float(torch.linalg.vector_norm(a))
    beta = norm(b)
    u = b / beta
    v = _adjoint(h, k, u)
    alpha = norm(v)
    v = v / alpha
    alphabar, zetabar = alpha, alpha * beta
    rho = rhobar = cbar = 1.0
    sbar = 0.0
    hv, hb, x = v.clone(), torch.zeros_like(v), torch.zeros_like(v)
    for _ in range(n_iter):
        u = _analysis(h, k, v) - alpha * u
        beta = norm(u)
        u = u / beta
        v = _adjoint(h, k, u) - beta * v
        alpha = norm(v)
        v = v / alpha
        old, rho = rho, math.hypot(alphabar, beta)
        c, s = alphabar / rho, beta / rho
        theta, alphabar = s * alpha, c * alpha
        oldbar, thetabar, t = rhobar, sbar * rho, cbar * rho
        rhobar = math.hypot(t, theta)
        cbar, sbar = t / rhobar, theta / rhobar
        zeta, zetabar = cbar * zetabar, -sbar * zetabar
        hb = hv - (thetabar * rho / (old * oldbar)) * hb
        x = x + (zeta / (rho * rhobar)) * hb
        hv = v - (theta / rho) * hv
    return x


def exact(case, seed):
    kind = case["kind"]
    st = prepare(case, seed)
    if kind == "serve":
        s, out = st["served"], []
        for c, (enu, azel), x in zip(s.shapes, s.geom, s.blocks):
            B, S = c["n_beams"], c["n_sb"]
            z = torch.zeros((B, S, HOP), dtype=torch.complex128, device=DEV)
            r = _exact_chain(c, x, enu, azel, z, z[:, :, :16],
                             DELAY + TAPS, False)
            out.append(dict(n_trig=None, snr=r["snr"].reshape(-1), best=None,
                            sample=None, beam=None, tec=None, trig_snr=None))
        return out
    if kind == "chain":
        p, o = st["p"], st["out"]
        r = _exact_chain(case, st["x"], st["enu"], st["azel"],
                         _as_c128(o["tail"]), _as_c128(o["hist"]),
                         keep=not case["group"])
        if case["group"]:
            del r["d"]
        return r
    k = _k(case)
    if kind == "beamform":
        return _real(_exact_beams(st["x"], _weights(st["enu"], st["azel"], k,
                                                    st["gain"])))
    if kind == "dedisperse":
        y, tail = _as_c128(st["y"]), _as_c128(st["tail"])
        d = torch.stack([torch.stack([
            _exact_dedisperse(y[b], tail[b], k, t) for t in st["tec"]])
            for b in range(case["n_beams"])])
        return dict(d=_real(d), tail=_real(y[:, :, case["n_t"] - HOP:]))
    if kind == "synthesize":
        d, hist = _as_c128(st["d"]), _as_c128(st["hist"])
        r = [_exact_series(d[i], hist[i], k, case["series"])
             for i in range(case["n_series"])]
        out = dict(emax=torch.stack([a[0] for a in r]),
                   psum=torch.stack([a[1] for a in r]),
                   hist=_real(d[:, :, case["n_t"] - 16:]))
        if case["series"]:
            out["series"] = torch.stack([a[2] for a in r])
        return out
    if kind == "two_stage":
        G, P = case["n_groups"], case["n_prelim"]
        grp, enu = st["group"], st["enu"]
        y1 = torch.cat([_exact_beams(st["x"], _weights(
            enu, st["prelim_azel"], k, np.repeat(grp == g, 2)))
            for g in range(G)])
        nb, npre = _unit(st["azel"]), _unit(st["prelim_azel"])
        pb = np.argmax(nb @ npre.T, axis=1)
        rg = np.stack([enu[grp == g].mean(0) for g in range(G)])
        cyc = _freq(k)[:, None, None] * ((nb - npre[pb]) @ rg.T)[None] / C_LIGHT
        c = torch.from_numpy(np.exp(-2j * np.pi * (cyc - np.floor(cyc)))).to(DEV)
        y = torch.stack([sum(c[:, b, g, None] * y1[g * P + pb[b]]
                             for g in range(G)) for b in range(len(pb))])
        return dict(y1=_real(y1), y=_real(y))
    if kind == "lsmr":
        y, kk = _as_c128(st["y"]), torch.from_numpy(k.astype(np.int64)).to(DEV)
        return torch.stack([_lsmr(_prototype(), kk, y[i], case["n_iter"])
                            for i in range(case["n_series"])])
    return None  # the station simulator's outputs are whole numbers
