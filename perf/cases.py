"""The workloads whose speed is tracked, each as one pass through the package's public entry points.

Sizes are those of the benchmark, the tests and the generators of this repository: up to 124 stations of two
channels, traces of 256 to 4096 samples (mostly 2048 and 4096), one to some thousands of candidate directions, the
30-80 MHz band at 200 MHz sampling, the 1 MHz / 5 degree complex128 pattern table in double precision and the
0.5 MHz / 1 degree complex64 table in single precision.

listed() names fixed cases, draw() gives further ones of the same ranges, prepare() holds what a program has before
the call (traces on the device, the loaded table, plans, output buffers and workspaces), run() is one pass, work()
the bytes and operations a pass cannot do without, exact() the same results from plain 64-bit torch.
"""
import numpy as np
import torch

from paper_1507_07733_amd import api, synth

DEV = "cuda"
C_M_PER_NS = 0.299792458
FIT_STEP = (3.0, 6.0)
MAX_OUT_BYTES = 12 << 30  # largest output of a drawn case
PLAN_FLAGS = api.AU_PLAN_GRAPH | api.AU_PLAN_PERSISTENT | api.AU_PLAN_XCD


def listed():
    return [
        # the plain call on a small event: ten stations, one direction; latency
        {"name": "event_fp64_10x2048", "kind": "event", "prec": 64, "s": 10, "n": 2048},
        # an ordinary event's traces for its fitted direction, short traces, single precision
        {"name": "event_fp32_57x1024", "kind": "event", "prec": 32, "s": 57, "n": 1024},
        # every station of the array for a full grid of candidates, double precision (the largest single call)
        {"name": "scan_fp64_124x4096x2048", "kind": "scan", "prec": 64, "s": 124, "n": 4096, "d": 2048},
        # a small grid of candidates for one ordinary event, as a served request asks for
        {"name": "scan_fp32_61x2048x64", "kind": "scan", "prec": 32, "s": 61, "n": 2048, "d": 64},
        # the batched workload: events of uneven size, 256 candidates each
        {"name": "plan_fp32_40ev_256dirs", "kind": "plan", "prec": 32, "events": 40, "d": 256, "s_max": 124,
         "n_min": 2048, "n_max": 4096},
        # the large batch: many full events with few candidates, inputs streaming through
        {"name": "plan_fp32_160ev_16dirs", "kind": "plan", "prec": 32, "events": 160, "d": 16, "s_max": 0,
         "n_min": 4096, "n_max": 4096},
        # a batch in double precision with every usual trace length
        {"name": "plan_fp64_32ev_64dirs", "kind": "plan", "prec": 64, "events": 32, "d": 64, "s_max": 124,
         "n_min": 1024, "n_max": 4096},
        # station timing of one event for many candidates: envelope maxima only, no traces kept
        {"name": "envelope_fp32_124x4096x512", "kind": "envelope", "prec": 32, "s": 124, "n": 4096, "d": 512},
        # coarse grid and four refinements of one event's direction
        {"name": "fit_fp64_124x4096x2048", "kind": "fit", "prec": 64, "s": 124, "n": 4096, "d": 2048, "levels": 4,
         "k": 5},
        # the iterative reconstruction of one event, its last traces kept
        {"name": "recon_fp64_124x4096", "kind": "recon", "prec": 64, "s": 124, "n": 4096},
        # the same for a batch of uneven events at once
        {"name": "recon_batch_fp32_96ev", "kind": "recon_batch", "prec": 32, "events": 96, "s_max": 124, "n": 4096},
        # a burst of requests to the server: host traces in, host results out
        {"name": "serve_fp32_16ev_57x2048", "kind": "serve", "prec": 32, "events": 16, "s": 57, "n": 2048, "d": 2},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["event", "scan", "scan", "plan", "plan", "envelope", "envelope", "fit", "recon", "recon_batch"])
    prec = rng.choice([32, 64])
    c = {"kind": kind, "prec": prec}
    s = rng.randint(3, 124)
    if kind == "event":
        c.update(s=s, n=rng.choice([256, 512, 1024, 2048, 4096]))
    elif kind in ("scan", "envelope"):
        n = rng.choice([256, 512, 1024, 2048, 2048, 4096, 4096])
        c.update(s=s, n=n, d=_log_int(rng, 3, 2048))
    elif kind == "plan":
        n_max = rng.choice([2048, 4096])
        d = _log_int(rng, 4, 256)
        per_event = (64 if prec == 32 else 128) * 2 * n_max * d * (prec // 32) * 4
        c.update(events=min(_log_int(rng, 8, 160), max(4, MAX_OUT_BYTES // per_event)), d=d,
                 s_max=rng.choice([0, 124]) if d <= 16 else 124, n_min=rng.choice([1024, 2048]), n_max=n_max)
    elif kind == "fit":
        c.update(s=s, n=rng.choice([2048, 4096]), d=_log_int(rng, 32, 2048), levels=rng.randint(1, 4), k=rng.choice([3, 5]))
    elif kind == "recon":
        c.update(s=s, n=rng.choice([2048, 4096]))
    else:
        c.update(events=_log_int(rng, 4, 96), s_max=124, n=rng.choice([2048, 4096]))
    return c


# ---------------------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------------------

_host_tables = {}
_tables = {}
_exact_tables = {}


def _host_table(prec):
    """(grid, table) of the array's antenna pattern: one fixed pattern per precision."""
    if prec not in _host_tables:
        g = synth.GRID_COARSE if prec == 64 else synth.GRID_FINE
        t = synth.pattern_table(g, cfg=0)
        _host_tables[prec] = (g, t if prec == 64 else t.astype(np.complex64))
    return _host_tables[prec]


def _table(prec):
    """The pattern loaded on the device: a program loads it once and keeps it for every event."""
    if prec not in _tables:
        _tables[prec] = api.load_pattern_table(*_host_table(prec))
    return _tables[prec]


def _dtype(prec):
    return torch.float64 if prec == 64 else torch.float32


def _event(prec, s, n):
    if prec == 64:
        return api.make_event(s, n)
    return api.make_event(s, n, prec=api.AU_PREC_FP32, trace_dtype=api.AU_F32)


def _traces(gen, s, n, prec, t0=None):
    """Traces [S][2][N]: unit noise and an in-band pulse of amplitude 5 to 20 at t0 (uniform where not given)."""
    if t0 is None:
        t0 = torch.rand(s, generator=gen, device=DEV, dtype=torch.float64) * n
    amp = 5 + 15 * torch.rand((s, 2, 1), generator=gen, device=DEV, dtype=torch.float64)
    kb = synth.band_bins(n)
    x = (2 * np.pi / n) * (torch.arange(n, device=DEV, dtype=torch.float64)[None, :] - t0[:, None])
    half = torch.sin(0.5 * x)
    small = half.abs() < 1e-12
    p = (torch.sin((float(kb[-1]) + 0.5) * x) - torch.sin((float(kb[0]) - 0.5) * x)) / (2 * torch.where(small, 1.0, half))
    p = torch.where(small, float(len(kb)), p) / len(kb)
    v = torch.randn((s, 2, n), generator=gen, device=DEV, dtype=torch.float64) + amp * p[:, None, :]
    return v.to(_dtype(prec)).contiguous()


def _plane_wave_traces(gen, r, pos, n, prec):
    """Traces whose pulses arrive as a plane wave from a random direction, centred in the trace."""
    zen = r.uniform(5.0, 55.0 if n >= 4096 else 40.0)
    t0 = n / 2.0 + synth.plane_wave_delays(pos, zen, r.uniform(0.0, 360.0))
    return _traces(gen, len(pos), n, prec, torch.from_numpy(t0).to(DEV))


def _dirs(r, d):
    """Candidate directions [D][2]: even in zenith up to 87 degrees, any azimuth."""
    out = np.empty((d, 2))
    out[:, 0] = (r.permutation(d) + r.random(d)) * (87.0 / d)
    out[:, 1] = r.random(d) * 360.0
    return out


def _inputs(case, seed):
    """Everything that is made from the seed: traces (device), directions and positions (host)."""
    r = np.random.default_rng([int(seed), 1507])
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 7919 + 7733)
    kind, prec = case["kind"], case["prec"]
    if kind == "event":
        return {"volt": _traces(gen, case["s"], case["n"], prec), "dirs": _dirs(r, 1)}
    if kind in ("scan", "envelope"):
        return {"volt": _traces(gen, case["s"], case["n"], prec), "dirs": _dirs(r, case["d"])}
    if kind in ("fit", "recon"):
        pos = synth.station_positions(case["s"])
        v = _plane_wave_traces(gen, r, pos, case["n"], prec)
        if kind == "recon":
            return {"volt": v, "pos": pos}
        return {"volt": v, "pos": pos, "dirs": _dirs(r, case["d"])}
    if kind == "plan":
        # sizes are the case's, whatever the seed: the same work in every state
        sizes = np.random.default_rng([case["events"], case["d"], case["n_max"]])
        lens = [n for n in (1024, 2048, 4096) if case["n_min"] <= n <= case["n_max"]]
        specs = []
        for _ in range(case["events"]):
            s = int(sizes.integers(3, case["s_max"] + 1)) if case["s_max"] else 124
            specs.append((s, int(sizes.choice(lens)), _dirs(r, case["d"])))
        return {"specs": specs, "volts": [_traces(gen, s, n, prec) for s, n, _ in specs]}
    if kind == "recon_batch":
        sizes = np.random.default_rng([case["events"], case["n"]])
        ns = [int(sizes.integers(3, case["s_max"] + 1)) for _ in range(case["events"])]
        pos = [synth.station_positions(s) for s in ns]
        return {"ns": ns, "pos": pos, "volts": [_plane_wave_traces(gen, r, p, case["n"], prec) for p in pos]}
    # serve: the requests' traces wait in pinned host memory
    volts = [_traces(gen, case["s"], case["n"], prec).cpu().pin_memory() for _ in range(case["events"])]
    return {"volts": volts, "dirs": [_dirs(r, case["d"]) for _ in volts]}


def prepare(case, seed):
    kind, prec = case["kind"], case["prec"]
    st = dict(_inputs(case, seed), case=case)
    tab = st["tab"] = _table(prec)
    dt = _dtype(prec)
    if kind in ("event", "scan", "envelope", "fit", "recon"):
        s, n = case["s"], case["n"]
        ev = st["ev"] = _event(prec, s, n)
        if kind in ("event", "scan", "envelope"):
            d = len(st["dirs"])
            st["work"] = torch.empty(api.workspace_bytes(tab, ev, d), dtype=torch.uint8, device=DEV)
            if kind == "event":
                st["out"] = torch.empty((s, 2, n), dtype=dt, device=DEV)
            elif kind == "scan":
                st["out"] = torch.empty((d, s, 2, n), dtype=dt, device=DEV)
        elif kind == "fit":
            b = api.direction_fit_workspace_bytes(tab, ev, len(st["dirs"]), case["levels"], case["k"])
            st["work"] = torch.empty(b, dtype=torch.uint8, device=DEV)
        else:
            st["work"] = torch.empty(api.reconstruct_workspace_bytes(tab, ev, 8), dtype=torch.uint8, device=DEV)
            st["out"] = torch.empty((s, 2, n), dtype=dt, device=DEV)
    elif kind == "plan":
        p64 = prec == 64
        plan = st["plan"] = api.Plan(tab, st["specs"], api.AU_PREC_FP64 if p64 else api.AU_PREC_FP32,
                                     api.AU_F64 if p64 else api.AU_F32,
                                     flags=PLAN_FLAGS | (api.AU_PLAN_FUSED if case["d"] <= 64 else 0))
        st["volt"] = torch.empty(plan.volt_elems, dtype=dt, device=DEV)
        for o, v in zip(plan.volt_offsets, st.pop("volts")):
            st["volt"][int(o):int(o) + v.numel()] = v.reshape(-1)
        st["out"] = torch.empty(plan.efield_elems, dtype=dt, device=DEV)
    elif kind == "recon_batch":
        st["ev"] = _event(prec, max(st["ns"]), case["n"])
        sz = np.array(st["ns"], dtype=np.int64) * 2 * case["n"]
        st["offsets"] = np.concatenate([[0], np.cumsum(sz)[:-1]])
        st["volt"] = torch.cat([v.reshape(-1) for v in st.pop("volts")])
        st["allpos"] = np.concatenate(st["pos"])
    else:
        st["server"] = api.Server(tab, 256 << 20, staging_bytes=64 << 20, max_inflight=64, n_streams=4, max_batch_events=16)
    return st


def run(state):
    c, tab = state["case"], state["tab"]
    kind = c["kind"]
    if kind == "event":
        z, a = state["dirs"][0]
        return api.unfold_event(tab, state["ev"], state["volt"], z, a, out=state["out"], work=state["work"])
    if kind == "scan":
        return api.unfold_direction_scan(tab, state["ev"], state["volt"], state["dirs"], out=state["out"], work=state["work"])
    if kind == "plan":
        state["plan"].run(state["volt"], state["out"])
        return state["out"]
    if kind == "envelope":
        peak, arg, _ = api.unfold_envelope_scan(tab, state["ev"], state["volt"], state["dirs"], work=state["work"])
        return {"peak": peak, "arg": arg}
    if kind == "fit":
        return api.direction_fit(tab, state["ev"], state["volt"], state["pos"], state["dirs"], levels=c["levels"], k=c["k"],
                                 step=FIT_STEP, work=state["work"])
    if kind == "recon":
        r = api.reconstruct(tab, state["ev"], state["volt"], state["pos"], max_iter=8, efield=state["out"], work=state["work"])
        return {"dirs": r.dirs, "times": r.times, "converged": r.converged, "efield": r.efield, "peak": r.peak}
    if kind == "recon_batch":
        rs = api.reconstruct_batch(tab, state["ev"], state["volt"], state["ns"], state["offsets"], state["allpos"], max_iter=8)
        return {"dirs": np.concatenate([r.dirs for r in rs]), "times": np.concatenate([r.times.ravel() for r in rs]),
                "passes": np.array([len(r.dirs) for r in rs]), "converged": np.array([int(r.converged) for r in rs])}
    sv = state["server"]
    tickets = [sv.submit(v, d) for v, d in zip(state["volts"], state["dirs"])]
    out = []
    for t in tickets:
        sv.wait(t)
        out.append(sv.result(t))
        sv.release(t)
    return out


def work(case):
    """Traces in and results out once; per station one forward transform, per (direction, station) the solve of the
    in-band bins and one inverse transform of the packed pair (two for an envelope), 5 N log2 N each."""
    kind, b = case["kind"], case["prec"] // 8

    def fwd(s, n):
        return {"bytes": 2.0 * n * b * s, "flops": 5.0 * n * np.log2(n) * s}

    def inv(s, n, d, out, transforms):
        return {"bytes": out * s * d, "flops": s * d * (transforms * 5.0 * n * np.log2(n) + 32.0 * len(synth.band_bins(n)))}

    parts = []
    if kind in ("event", "scan", "serve"):
        s, n, d = case["s"] * case.get("events", 1), case["n"], case.get("d", 1)
        parts = [fwd(s, n), inv(s, n, d, 2.0 * n * b, 1)]
    elif kind in ("envelope", "fit"):
        s, n = case["s"], case["n"]
        d = case["d"] + case.get("levels", 0) * case.get("k", 0) ** 2
        parts = [fwd(s, n), inv(s, n, d, 3.0 * (b + 4) if kind == "envelope" else 16.0 / s, 2)]
    elif kind == "recon":
        s, n = case["s"], case["n"]
        parts = [fwd(s, n), inv(s, n, 1, 2.0 * n * b, 2), inv(s, n, 1, 12.0, 2)]
    elif kind == "recon_batch":
        sizes = np.random.default_rng([case["events"], case["n"]])
        s = sum(int(sizes.integers(3, case["s_max"] + 1)) for _ in range(case["events"]))
        parts = [fwd(s, case["n"]), inv(s, case["n"], 2, 4.0, 2)]
    else:
        sizes = np.random.default_rng([case["events"], case["d"], case["n_max"]])
        lens = [n for n in (1024, 2048, 4096) if case["n_min"] <= n <= case["n_max"]]
        for _ in range(case["events"]):
            s = int(sizes.integers(3, case["s_max"] + 1)) if case["s_max"] else 124
            n = int(sizes.choice(lens))
            parts += [fwd(s, n), inv(s, n, case["d"], 2.0 * n * b, 1)]
    return {k: float(sum(p[k] for p in parts)) for k in ("bytes", "flops")}


# ---------------------------------------------------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------------------------------------------------


class _Exact:
    """In-band field spectra, traces and envelopes of one event in double precision, by plain torch."""

    def __init__(self, prec, volt):
        self.g, t = _host_table(prec)
        if prec not in _exact_tables:
            _exact_tables[prec] = torch.from_numpy(t).to(DEV).to(torch.complex128)
        self.t = _exact_tables[prec]
        self.n = volt.shape[-1]
        self.bins = torch.from_numpy(synth.band_bins(self.n)).to(DEV)
        self.x = torch.fft.fft(volt.to(torch.float64))[..., self.bins]  # [S][2][K]

    def response(self, dirs):
        """H [2][2][K][D], linear in azimuth, zenith and frequency between the nodes."""
        g = self.g
        zen, az = torch.as_tensor(dirs[:, 0], device=DEV), torch.as_tensor(dirs[:, 1], device=DEV)
        u = ((zen - g.zen0_deg) / g.dzen_deg).clamp(0, g.n_zen - 1)
        iz = u.floor().clamp(max=g.n_zen - 2).long()
        w = torch.remainder(az - g.az0_deg, 360.0) / g.daz_deg
        ia = w.floor().long()
        ta, ia = w - ia, ia % g.n_az
        ja, tz = (ia + 1) % g.n_az, u - iz
        num = self.bins * synth.FS_HZ - g.f0_hz * self.n
        jf = (num // (self.n * g.df_hz)).clamp(max=g.n_freq - 2)
        tf = (num - jf * self.n * g.df_hz).double() / float(self.n * g.df_hz)
        lo, hi = int(jf.min()), int(jf.max()) + 2
        t = self.t[:, :, lo:hi]
        a = t[..., iz, ia] * (1 - ta) + t[..., iz, ja] * ta
        b = t[..., iz + 1, ia] * (1 - ta) + t[..., iz + 1, ja] * ta
        s = a * (1 - tz) + b * tz                                    # [2][2][F][D]
        f = tf[None, None, :, None]
        return s[:, :, jf - lo] * (1 - f) + s[:, :, jf - lo + 1] * f

    def spectra(self, dirs):
        """In-band field spectra [D][S][2][K]."""
        h = self.response(dirs).permute(3, 0, 1, 2)[:, None]         # [D][1][2][2][K]
        det = h[:, :, 0, 0] * h[:, :, 1, 1] - h[:, :, 0, 1] * h[:, :, 1, 0]
        x0, x1 = self.x[None, :, 0], self.x[None, :, 1]
        return torch.stack([(h[:, :, 1, 1] * x0 - h[:, :, 0, 1] * x1) / det,
                            (h[:, :, 0, 0] * x1 - h[:, :, 1, 0] * x0) / det], dim=2)

    def _chunk(self):
        return max(1, (1 << 27) // (self.x.shape[0] * 2 * self.n))

    def field(self, dirs, out=None):
        """Traces [D][S][2][N]."""
        d, c = len(dirs), self._chunk()
        if out is None:
            out = torch.empty((d, self.x.shape[0], 2, self.n), dtype=torch.float64, device=DEV)
        for i in range(0, d, c):
            e = self.spectra(dirs[i:i + c])
            z = torch.zeros(e.shape[:-1] + (self.n // 2 + 1,), dtype=e.dtype, device=DEV)
            z[..., self.bins] = e
            out[i:i + c] = torch.fft.irfft(z, n=self.n)
        return out

    def envelope(self, dirs):
        """(peak [D][S][3], sample [D][S][3]) of the theta, phi and total-field envelopes."""
        pk, at = [], []
        c = self._chunk()
        for i in range(0, len(dirs), c):
            e = self.spectra(dirs[i:i + c])
            z = torch.zeros(e.shape[:-1] + (self.n,), dtype=e.dtype, device=DEV)
            z[..., self.bins] = 2 * e
            a = torch.fft.ifft(z)
            p = a.real.square() + a.imag.square()                     # [D][S][2][N]
            p = torch.cat([p, p.sum(dim=2, keepdim=True)], dim=2)
            m, j = p.max(dim=-1)
            pk.append(m.sqrt())
            at.append(j)
        return torch.cat(pk), torch.cat(at)


def _exact_fit(case, volt, pos, dirs, step):
    """Scores of every candidate, coarse ones first, then each level's grid around the best so far."""
    x = _Exact(case["prec"], volt)
    k, levels, chi2, power, grids = case["k"], case["levels"], [], [], []
    for lv in range(levels + 1):
        peak, arg = x.envelope(dirs)
        zr, ar = np.deg2rad(dirs[:, :1]), np.deg2rad(dirs[:, 1:])
        tau = -(np.sin(zr) * np.cos(ar) * pos[:, 0] + np.sin(zr) * np.sin(ar) * pos[:, 1]) / C_M_PER_NS
        r = arg[:, :, 2].cpu().numpy() * (1e9 / synth.FS_HZ) - tau
        c = ((r - r.mean(axis=1, keepdims=True)) ** 2).sum(axis=1)
        chi2.append(c)
        power.append(peak[:, :, 2].square().sum(dim=1).cpu().numpy())
        centre = dirs[int(c.argmin())]
        if lv < levels:
            o = (np.arange(k) - 0.5 * (k - 1)) * 2.0 ** -(lv + 1)
            z = np.clip(centre[0] + o * step[0], 0.0, 90.0)
            dirs = np.stack([np.repeat(z, k), np.tile((centre[1] + o * step[1]) % 360.0, k)], axis=1)
            grids.append(dirs)
    return {"result": centre, "best": None, "chi2": np.concatenate(chi2), "power": np.concatenate(power),
            "level_dirs": np.array(grids)}


def _plane_fit(t_ns, pos):
    a = np.stack([np.ones(len(pos)), pos[:, 0], pos[:, 1]], axis=1)
    _, p, q = np.linalg.lstsq(a, t_ns, rcond=None)[0]
    nx, ny = -C_M_PER_NS * p, -C_M_PER_NS * q
    return np.array([np.degrees(np.arcsin(min(1.0, np.hypot(nx, ny)))), np.degrees(np.arctan2(ny, nx)) % 360.0])


def _exact_recon(prec, volt, pos, max_iter=8):
    """(directions [K][2], exact event) of the reconstruction loop."""
    x = _Exact(prec, volt)
    v = volt.to(torch.float64)
    times = (v[:, 0].square() + v[:, 1].square()).argmax(dim=-1).cpu().numpy()
    dirs = []
    for _ in range(max_iter):
        dirs.append(_plane_fit(times * (1e9 / synth.FS_HZ), pos))
        new = x.envelope(np.array(dirs[-1:]))[1][0, :, 2].cpu().numpy()
        if np.array_equal(new, times):
            break
        times = new
    return np.array(dirs), x


def exact(case, seed):
    kind, prec = case["kind"], case["prec"]
    st = _inputs(case, seed)
    if kind == "event":
        return _Exact(prec, st["volt"]).field(st["dirs"])[0]
    if kind == "scan":
        return _Exact(prec, st["volt"]).field(st["dirs"])
    if kind == "envelope":
        return {"peak": _Exact(prec, st["volt"]).envelope(st["dirs"])[0], "arg": None}
    if kind == "plan":
        size = [len(d) * s * 2 * n for s, n, d in st["specs"]]
        out = torch.empty(sum(size), dtype=torch.float64, device=DEV)
        o = 0
        for (s, n, d), v, k in zip(st["specs"], st["volts"], size):
            _Exact(prec, v).field(d, out[o:o + k].view(len(d), s, 2, n))
            o += k
        return out
    if kind == "recon":
        dirs, x = _exact_recon(prec, st["volt"], st["pos"])
        return {"dirs": dirs, "times": None, "converged": None, "efield": x.field(dirs[-1:])[0],
                "peak": x.envelope(dirs[-1:])[0][0]}
    if kind == "recon_batch":
        return {"dirs": np.concatenate([_exact_recon(prec, v, p)[0] for v, p in zip(st["volts"], st["pos"])]),
                "times": None, "passes": None, "converged": None}
    if kind == "fit":
        return _exact_fit(case, st["volt"], st["pos"], st["dirs"], FIT_STEP)
    return [_Exact(prec, v.to(DEV)).field(d).cpu().numpy() for v, d in zip(st["volts"], st["dirs"])]
