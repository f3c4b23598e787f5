"""The work that this framework's time goes into, as callable cases.

A case is a plain dict.  Its `kind` says which program it stands for:

  steps     ctx.step() of one running system: the product path of every
            simulation (captured middle steps, rebuilds decided on the
            device), from the smallest box, where launches and latency are
            all, to the bulk liquid;
  batch     ctx.step() of an uneven ensemble of LJ liquids and bead-spring
            melts in one context;
  evaluate  forces, energies and virial of a configuration that has no list
            yet (Morton sort, cell list, list build, force pass, sums): what a
            program does with each frame of a trajectory;
  exchange  one subdomain's step around a ghost exchange whose transport is
            elsewhere: update and pack the send list, unpack what came, local
            forces;
  reselect  the same at a rebuild: select and pack anew, unpack the new
            layer, build the list, local forces.

Liquids are melts (a small fcc box run above its melting point here in plain
torch, repeated through the box, then random vacancies and fresh velocities),
so that tiles, cells and rows have the spread they have in a running
simulation; the DPD fluid and the polymer melts are the repository's own
recipes.
"""
import math

import numpy as np
import torch

from paper_1412_3387_amd import binding as B
from paper_1412_3387_amd import inputs

LIQUID_T = 0.65   # where the bulk liquid started at T = 1.2 from the lattice settles
WEAK_DENSITY = 6.0 * 0.2 / math.pi  # packing fraction 0.2, the weak-scaling fluid
# fcc cells per side of the LJ boxes: each is b k with b <= 10, so that a
# melted box of b^3 cells fills it when repeated k times per axis
SIDES = (6, 7, 8, 9, 10, 12, 14, 16, 18, 20, 24, 28, 30, 32, 36, 40, 48, 50, 56, 64, 72, 80)
SUB_SIDES = (24, 30, 36, 48, 60, 72)  # fcc cells per side of a box cut into 3 x 3 x 3 subdomains


def listed():
    return [
        # the parity-sized liquid: 63 tiles, every step is launch latency
        dict(name="lj_4k", kind="steps", fluid="lj", n=4000, fp64=False, steps=50, log=0),
        # one GPU's share of the weak-scaling runs: NVT, logged every 10 steps
        dict(name="nvt_32k_log", kind="steps", fluid="weak", n=32000, fp64=False, steps=50, log=10),
        # an ordinary liquid in full precision, an odd size
        dict(name="lj_255k_fp64", kind="steps", fluid="lj", n=254999, fp64=True, steps=20, log=0),
        # the bulk liquid of the headline benchmark
        dict(name="lj_2m", kind="steps", fluid="lj", n=2000000, fp64=False, steps=20, log=0),
        # the DPD fluid of the benchmark, and a small one in full precision
        dict(name="dpd_1m", kind="steps", fluid="dpd", n=1000000, fp64=False, steps=10, log=0),
        dict(name="dpd_100k_fp64", kind="steps", fluid="dpd", n=100003, fp64=True, steps=10, log=0),
        # one bead-spring melt: FENE bonds, WCA, exclusions
        dict(name="melt_50k", kind="steps", fluid="melt", n=50000, fp64=False, steps=20, log=0),
        # a quarter of the benchmark's ensemble
        dict(name="batch_64", kind="batch", n_lj=32, n_poly=32, largest=20000, fp64=False, steps=20),
        # frames evaluated one by one
        dict(name="frame_498k_fp64", kind="evaluate", fluid="lj", n=497999, fp64=True),
        dict(name="frame_31k", kind="evaluate", fluid="lj", n=31333, fp64=False),
        # the strong-scaling subdomain between rebuilds, and at one
        dict(name="subdomain_32k", kind="exchange", n=864000, fp64=False),
        dict(name="subdomain_32k_select", kind="reselect", n=864000, fp64=False),
    ]


def _lj_n(rng, lo, hi):
    """A full fcc lattice's size, or that less up to 2 % vacancies."""
    m = rng.choice([s for s in SIDES if lo <= 4 * s ** 3 <= hi])
    return 4 * m ** 3 - (rng.randrange(1, max(2, 4 * m ** 3 // 50)) if rng.random() < 0.8 else 0)


def _log_n(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(("steps", "steps", "steps", "steps", "batch", "evaluate", "evaluate", "exchange", "reselect"))
    fp64 = rng.random() < 0.4
    if kind == "steps":
        fluid = rng.choice(("lj", "lj", "weak", "dpd", "melt"))
        if fluid in ("lj", "weak"):
            n = _lj_n(rng, 860, 1100000)
            return dict(kind=kind, fluid=fluid, n=n, fp64=fp64, steps=20 if n > 200000 else 50,
                        log=rng.choice((0, 0, 10)))
        if fluid == "dpd":
            return dict(kind=kind, fluid=fluid, n=_log_n(rng, 3000, 600000), fp64=fp64, steps=10, log=0)
        return dict(kind=kind, fluid=fluid, n=50 * _log_n(rng, 20, 2500), fp64=fp64, steps=20, log=0)
    if kind == "batch":
        return dict(kind=kind, n_lj=rng.randrange(1, 33), n_poly=rng.randrange(1, 33),
                    largest=_log_n(rng, 3000, 20000), fp64=fp64, steps=20)
    if kind == "evaluate":
        return dict(kind=kind, fluid="lj", n=_lj_n(rng, 860, 1100000), fp64=fp64)
    n = 4 * rng.choice(SUB_SIDES) ** 3
    return dict(kind=kind, n=n - rng.randrange(1, n // 50), fp64=fp64)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _melted_cell(b, L, T, seed):
    """Positions of 4 b^3 particles in a cube of side L: an fcc lattice run
    for 250 velocity-Verlet steps of 0.005 with truncated LJ forces, held at
    about 1.4 (the fluid's T if higher) and cooled to T at the end."""
    n = 4 * b ** 3
    rng = np.random.default_rng([seed, 1])
    dev = _device()
    x = torch.as_tensor(inputs.fcc_sites(b, L) + rng.uniform(-0.05, 0.05, (n, 3)), device=dev)
    v = torch.as_tensor(inputs.maxwell_velocities(n, max(1.4, T), int(rng.integers(1 << 30))), device=dev)
    eye = torch.arange(n, device=dev)
    rc = min(2.5, 0.49 * L)

    def force():
        r2 = torch.zeros((n, n), dtype=torch.float64, device=dev)
        for a in range(3):
            d = x[:, None, a] - x[None, :, a]
            d -= L * torch.round(d / L)
            r2 += d * d
        r2[eye, eye] = 4.0 * rc * rc
        i2 = 1.0 / r2
        s6 = i2 * i2 * i2
        ff = torch.where(r2 < rc * rc, 24.0 * s6 * (2.0 * s6 - 1.0) * i2, torch.zeros_like(r2))
        # sum_j ff (x_i - x_j), image by image
        out = torch.empty_like(x)
        for a in range(3):
            d = x[:, None, a] - x[None, :, a]
            out[:, a] = (ff * (d - L * torch.round(d / L))).sum(1)
        return out

    f = force()
    for s in range(250):
        v = v + 0.0025 * f
        x = x + 0.005 * v
        x = x - L * torch.floor(x / L)
        f = force()
        v = v + 0.0025 * f
        if s % 10 == 9:
            want = max(1.4, T) if s < 180 else T
            v = v * torch.sqrt(want / ((v * v).sum() / (3 * n - 3)))
    return x.cpu().numpy()


def _liquid(n, density, T, seed):
    """(pos, vel, L) of an LJ liquid of n particles."""
    m = next(s for s in SIDES if 4 * s ** 3 >= n)
    b = next(q for q in range(10, 5, -1) if m % q == 0)
    k = m // b
    L = (n / density) ** (1.0 / 3.0)
    cell = _melted_cell(b, L / k, T, seed)
    g = np.arange(k, dtype=np.float64) * (L / k)
    gz, gy, gx = np.meshgrid(g, g, g, indexing="ij")
    shifts = np.stack([gx.ravel(), gy.ravel(), gz.ravel()], axis=1)
    pos = (shifts[:, None, :] + cell[None, :, :]).reshape(-1, 3)
    rng = np.random.default_rng([seed, 2])
    if pos.shape[0] > n:
        keep = np.ones(pos.shape[0], dtype=bool)
        keep[rng.choice(pos.shape[0], pos.shape[0] - n, replace=False)] = False
        pos = pos[keep]
    pos = pos + rng.uniform(-0.01, 0.01, pos.shape)
    Lv = np.full(3, L)
    return inputs.wrap(pos, Lv), inputs.maxwell_velocities(n, T, seed + 3), Lv


def _system(fluid, n, seed):
    if fluid == "lj":
        pos, vel, L = _liquid(n, inputs.LJ_DENSITY, LIQUID_T, seed)
    elif fluid == "weak":
        pos, vel, L = _liquid(n, WEAK_DENSITY, 1.2, seed)
    elif fluid == "dpd":
        s = inputs.dpd_fluid(n, seed + 1, seed + 2)
        pos, vel, L = s.pos, s.vel, s.L
    else:
        s = inputs.polymer_melt(n // 50, seed + 1)
        return dict(pos=s.pos, vel=s.vel, L=s.L, tag=s.tag, bonds=s.bonds)
    return dict(pos=pos, vel=vel, L=L, tag=np.arange(n, dtype=np.int32))


def _params(fluid, fp64):
    prec = B.FP64 if fp64 else B.MIXED
    if fluid == "lj":
        return B.ModelParams(precision=prec, r_cut=2.5, r_buff=0.4, dt=0.005, sort_period=500)
    if fluid == "weak":
        return B.ModelParams(precision=prec, r_cut=3.0, r_buff=0.4, dt=0.002, sort_period=500, integrator=B.NVT,
                             nvt_T0=1.2, nvt_tau=0.5)
    if fluid == "dpd":
        return B.ModelParams(precision=prec, pair=B.PAIR_DPD, r_cut=1.0, r_buff=0.5, dt=0.02, dpd_seed=33,
                             sort_period=20)
    return B.ModelParams(precision=prec, pair=B.PAIR_WCA, bond_cap=2, dt=0.005, sort_period=500)


def _ensemble(case, seed):
    """[(fluid, system)]: LJ liquids of 500 particles and up, and melts of 20
    chains and up, of sizes that the case alone decides."""
    rng = np.random.default_rng([case["n_lj"], case["n_poly"], case["largest"]])
    out = []
    for k in range(case["n_lj"]):
        n = int(rng.integers(500, case["largest"] + 1))
        s = inputs.lj_fluid(n, seed + 10 * k, seed + 10 * k + 1, seed + 10 * k + 2)
        out.append(("lj", dict(pos=s.pos, vel=s.vel, L=s.L, tag=s.tag)))
    for k in range(case["n_poly"]):
        c = int(rng.integers(20, case["largest"] // 50 + 1))
        out.append(("melt", _system("melt", 50 * c, seed + 5000 + 10 * k)))
    return out


SUB_W, SUB_MARGIN = 2.9, 0.25  # ghost width (r_cut + r_buff) and the frame's room beyond it


def _subdomain(case, seed):
    """Subdomain 0 of a periodic liquid cut 3 x 3 x 3: its locals, the records
    its neighbours send it, and its frame."""
    pos, vel, L = _liquid(case["n"], inputs.LJ_DENSITY, LIQUID_T, seed)
    side = L[0] / 3.0
    local = np.all(pos < side, axis=1)
    # the image nearest the subdomain's centre decides what lies in the layer
    near = pos - L * np.rint((pos - 0.5 * side) / L)
    ghost = np.all((near >= -SUB_W) & (near < side + SUB_W), axis=1) & ~local
    rows, gh = np.nonzero(local)[0], np.nonzero(ghost)[0]
    rec = np.zeros(gh.size, dtype=[("x", "f8", 3), ("tag", "i4"), ("pad", "i4")])
    rec["x"] = pos[gh]
    rec["tag"] = gh
    frame = side + 2 * (SUB_W + SUB_MARGIN)
    return dict(pos=pos[rows], vel=vel[rows], tag=rows.astype(np.int32), L=np.full(3, frame),
                lo=np.full(3, -SUB_W - SUB_MARGIN), periodic=(0, 0, 0),
                n_cap=int(1.2 * inputs.LJ_DENSITY * frame ** 3) + 64), near[gh], gh.astype(np.int32), rec, L, side


def prepare(case, seed):
    seed = 7 + 100003 * (seed % 20000)
    if case["kind"] == "batch":
        ens = _ensemble(case, seed)
        ctx = B.Context([_params(f, case["fp64"]) for f, _ in ens], [s for _, s in ens])
        ctx.build_nlist(True)
        return dict(kind="steps", ctx=ctx, t=0, steps=case["steps"], log=0)
    if case["kind"] in ("steps", "evaluate"):
        ctx = B.Context([_params(case["fluid"], case["fp64"])], [_system(case["fluid"], case["n"], seed)])
        if case["kind"] == "evaluate":
            return dict(kind="evaluate", ctx=ctx)
        ctx.build_nlist(True)
        return dict(kind="steps", ctx=ctx, t=0, steps=case["steps"], log=case["log"])
    sysd, _, gh, rec, L, side = _subdomain(case, seed)
    ctx = B.Context([B.ModelParams(precision=B.FP64 if case["fp64"] else B.MIXED, nlist_cap=160)], [sysd])
    dev = ctx.device
    cap = case["n"] // 13
    st = dict(kind=case["kind"], ctx=ctx, lo=np.zeros(3), hi=np.full(3, side), box=L, n_recv=int(gh.size), cap=cap,
              recv=torch.as_tensor(rec.view(np.uint8).reshape(-1).copy(), device=dev),
              send=torch.zeros(32 * cap, dtype=torch.uint8, device=dev),
              counts=torch.zeros(26, dtype=torch.int32, device=dev),
              offsets=torch.zeros(26, dtype=torch.int32, device=dev))
    _ghosts(st, B.GHOST_SELECT)
    ctx.build_nlist(True)
    return st


def _ghosts(st, mode):
    fields = B.FIELD_POS | B.FIELD_TAG
    st["ctx"].pack_ghosts(0, st["lo"], st["hi"], SUB_W, mode, fields, st["send"], st["cap"], st["counts"],
                          st["offsets"])
    st["ctx"].unpack_ghosts(0, st["recv"], st["n_recv"], fields, mode, st["box"])


def run(st):
    ctx = st["ctx"]
    if st["kind"] == "steps":
        ctx.step(st["t"], st["steps"], st["log"])
        st["t"] += st["steps"]
        out = dict(pos=ctx.pos, vel=ctx.vel, force=ctx.force, tag=ctx.tag)
        if st["log"]:
            out["log"] = ctx.thermo_log(st["steps"] + 1)
        return out
    if st["kind"] == "evaluate":
        ctx.build_nlist(True)
        ctx.compute_forces(0, B.ENERGY | B.VIRIAL)
        return dict(force=ctx.force, pos=ctx.pos, tag=ctx.tag, thermo=ctx.thermo())
    if st["kind"] == "exchange":
        _ghosts(st, B.GHOST_UPDATE)
    else:
        _ghosts(st, B.GHOST_SELECT)
        ctx.build_nlist(True)
    ctx.compute_forces(0, 0)
    return dict(force=ctx.force, pos=ctx.pos, tag=ctx.tag, send=st["send"], counts=st["counts"],
                offsets=st["offsets"])


# mean neighbours inside the cut-off, and floating-point operations of one
# listed pair inside it (separation, r^2, pair term, sums)
def _inside(fluid):
    if fluid == "lj":
        return 4.0 / 3.0 * math.pi * 2.5 ** 3 * inputs.LJ_DENSITY, 27
    if fluid == "weak":
        return 4.0 / 3.0 * math.pi * 27.0 * WEAK_DENSITY, 27
    if fluid == "dpd":
        return 4.0 / 3.0 * math.pi * inputs.DPD_DENSITY, 80
    return 4.0 / 3.0 * math.pi * math.sqrt(2.0) * inputs.POLYMER_DENSITY + 2.0, 27


def work(case):
    """Per step and particle the state (x, v: 3 doubles each) read and
    written once, and every pair inside the cut-off computed once."""
    if case["kind"] == "batch":
        # the ensemble's mean sizes
        n = case["n_lj"] * (500 + case["largest"]) / 2 + case["n_poly"] * 50 * (20 + case["largest"] // 50) / 2
        return {"bytes": 96.0 * n * case["steps"],
                "flops": 0.5 * n * case["steps"] * sum(0.5 * p * q for p, q in (_inside("lj"), _inside("melt")))}
    if case["kind"] == "steps":
        p, q = _inside(case["fluid"])
        return {"bytes": 96.0 * case["n"] * case["steps"], "flops": 0.5 * p * q * case["n"] * case["steps"]}
    p, q = _inside("lj")
    f = 32 if case["fp64"] else 16
    if case["kind"] == "evaluate":
        return {"bytes": (24.0 + f) * case["n"], "flops": 0.5 * p * q * case["n"]}
    n = case["n"] / 27.0
    side = (n / inputs.LJ_DENSITY) ** (1.0 / 3.0)
    ghosts = inputs.LJ_DENSITY * ((side + 2 * SUB_W) ** 3 - side ** 3)
    # locals read once, a record packed and one unpacked per ghost
    return {"bytes": (24.0 + f) * n + 2 * 2 * 32.0 * ghosts, "flops": 0.5 * p * q * n}


# ---------------------------------------------------------------------------
# what the cases compute, in 64 bits with plain torch
# ---------------------------------------------------------------------------

class _Pairs:
    """Pairs (i < j) within reach of each other, from a cell grid per system."""

    def __init__(self, systems, fluids, rc, skin, dev):
        # per particle: system, box, first cell and cells per axis
        n = [s["pos"].shape[0] for s in systems]
        self.dev, self.skin = dev, skin
        sid = np.repeat(np.arange(len(n)), n)
        L = np.array([s["L"] for s in systems], dtype=np.float64)
        lo = np.array([s.get("lo", np.zeros(3)) for s in systems], dtype=np.float64)
        reach = np.array(rc) + skin
        bins = np.maximum(1, np.floor(L / reach[:, None]).astype(np.int64))
        first = np.concatenate([[0], np.cumsum(bins.prod(1))])
        per = np.array([s.get("periodic", (1, 1, 1)) for s in systems], dtype=bool)
        t = lambda a: torch.as_tensor(a, device=dev)  # noqa: E731
        self.ncell = int(first[-1])
        self.L, self.lo, self.bins, self.per = t(L)[t(sid)], t(lo)[t(sid)], t(bins)[t(sid)], t(per)[t(sid)]
        self.first, self.reach2 = t(first[:-1])[t(sid)], t(reach ** 2)[t(sid)]
        # tag pairs that are bonded take no part
        self.excluded = None
        base, keys = 0, []
        self.total = int(sum(n))
        self.bond = None
        for s, m in zip(systems, n):
            if s.get("bonds") is not None:
                b = np.asarray(s["bonds"], dtype=np.int64) + base
                keys.append(np.stack([b.min(1), b.max(1)]))
            base += m
        if keys:
            b = np.concatenate(keys, axis=1)
            self.bond = t(b)
            self.excluded = torch.sort(t(b[0] * self.total + b[1]))[0]

    def image(self, d, i):
        L = self.L[i]
        return torch.where(self.per[i], d - L * torch.round(d / L), d)

    def build(self, x):
        n, dev = x.shape[0], self.dev
        c = torch.minimum(((x - self.lo) / self.L * self.bins).floor().long().clamp(min=0), self.bins - 1)
        cid = self.first + (c[:, 2] * self.bins[:, 1] + c[:, 1]) * self.bins[:, 0] + c[:, 0]
        order = torch.argsort(cid)
        count = torch.bincount(cid, minlength=self.ncell)
        start = torch.cumsum(count, 0) - count
        cap, me = int(count.max()), torch.arange(n, device=dev)
        ii, jj = [], []
        for o in range(27):
            off = torch.tensor([o % 3 - 1, o // 3 % 3 - 1, o // 9 - 1], device=dev)
            # an axis of two cells has one other cell, an axis of one none
            ok = ((self.bins >= 3) | ~self.per | (off == 0) | ((self.bins == 2) & (off == 1))).all(1)
            q = c + off
            inside = ((q >= 0) & (q < self.bins)) | self.per
            ok &= inside.all(1)
            q = torch.where(self.per, torch.remainder(q, self.bins), q.clamp(min=0))
            q = torch.minimum(q, self.bins - 1)
            nc = self.first + (q[:, 2] * self.bins[:, 1] + q[:, 1]) * self.bins[:, 0] + q[:, 0]
            cnt = torch.where(ok, count[nc], torch.zeros_like(nc))
            st = start[nc]
            for k in range(cap):
                i = me[cnt > k]
                if i.numel() == 0:
                    break
                j = order[st[i] + k]
                keep = j > i
                i, j = i[keep], j[keep]
                d = self.image(x[i] - x[j], i)
                keep = (d * d).sum(1) < self.reach2[i]
                ii.append(i[keep])
                jj.append(j[keep])
        self.i, self.j, self.x0 = torch.cat(ii), torch.cat(jj), x.clone()
        if self.excluded is not None and self.excluded.numel():
            key = self.i * self.total + self.j
            at = torch.searchsorted(self.excluded, key).clamp(max=self.excluded.numel() - 1)
            keep = self.excluded[at] != key
            self.i, self.j = self.i[keep], self.j[keep]

    def update(self, x):
        if hasattr(self, "x0"):
            d = x - self.x0
            d = torch.where(self.per, d - self.L * torch.round(d / self.L), d)
            if 2.0 * math.sqrt(float((d * d).sum(1).max())) < self.skin:
                return
        self.build(x)


def _philox(a, b, seed, step):
    """First word of Philox4x32-10 of counter (a, b, 0, 0), key (seed, step)."""
    def mul(m, v):
        t = m * (v & 0xFFFF)
        u = m * (v >> 16) + (t >> 16)
        return u >> 16, ((u & 0xFFFF) << 16) | (t & 0xFFFF)
    c0, c1, c2, c3 = a, b, torch.zeros_like(a), torch.zeros_like(a)
    k0, k1 = seed, step & 0xFFFFFFFF
    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c0)
        h1, l1 = mul(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c0


def _lj(r2, shift):
    i2 = 1.0 / r2
    s6 = i2 * i2 * i2
    return 24.0 * s6 * (2.0 * s6 - 1.0) * i2, 4.0 * s6 * (s6 - 1.0) - shift


class _Model:
    """Forces, energies and virial of the concatenated systems."""

    def __init__(self, systems, fluids, dev, skin):
        self.fluids, self.dev = fluids, dev
        rcs = {"lj": 2.5, "weak": 3.0, "dpd": 1.0, "melt": 2.0 ** (1.0 / 6.0)}
        rc = np.array([rcs[f] for f in fluids])
        self.pairs = _Pairs(systems, fluids, rc, skin, dev)
        n = [s["pos"].shape[0] for s in systems]
        sh = [-1.0 if f == "melt" else 4.0 * (r ** -12 - r ** -6) for f, r in zip(fluids, rc)]
        sid = torch.as_tensor(np.repeat(np.arange(len(n)), n), device=dev)
        self.rc2 = torch.as_tensor(rc ** 2, device=dev)[sid]
        self.shift = torch.as_tensor(np.array(sh), device=dev)[sid]
        self.dpd = fluids[0] == "dpd"

    def __call__(self, x, v, t):
        P = self.pairs
        P.update(x)
        F, e = torch.zeros_like(x), torch.zeros(x.shape[0], dtype=x.dtype, device=x.device)
        W = 0.0
        for q in range(0, P.i.numel(), 1 << 25):
            i, j = P.i[q:q + (1 << 25)], P.j[q:q + (1 << 25)]
            d = P.image(x[i] - x[j], i)
            r2 = (d * d).sum(1)
            m = (r2 < self.rc2[i]) & (r2 > 0)
            i, j, d, r2 = i[m], j[m], d[m], r2[m]
            if self.dpd:
                r = torch.sqrt(r2)
                w = 1.0 - r
                rv = (d * (v[i] - v[j])).sum(1) / r
                bits = _philox(i, j, 33, t) >> 8
                theta = math.sqrt(3.0) * (2.0 * bits.double() / 16777216.0 - 1.0)
                ff = (25.0 * w - 4.5 * w * w * rv + math.sqrt(9.0) * w * theta / math.sqrt(0.02)) / r
                u = 12.5 * w * w
            else:
                ff, u = _lj(r2, self.shift[i])
            W += float((ff * r2).sum())
            f = ff[:, None] * d
            F.index_add_(0, i, f)
            F.index_add_(0, j, -f)
            e.index_add_(0, i, 0.5 * u)
            e.index_add_(0, j, 0.5 * u)
        if P.bond is not None:
            i, j = P.bond
            d = P.image(x[i] - x[j], i)
            r2 = (d * d).sum(1)
            g = 1.0 - r2 / 2.25
            fl, ul = _lj(r2, -1.0)
            near = r2 < 2.0 ** (1.0 / 3.0)
            zero = torch.zeros_like(r2)
            ff = -30.0 / g + torch.where(near, fl, zero)
            u = -0.5 * 30.0 * 2.25 * torch.log(g) + torch.where(near, ul, zero)
            W += float((ff * r2).sum())
            f = ff[:, None] * d
            F.index_add_(0, i, f)
            F.index_add_(0, j, -f)
            e.index_add_(0, i, 0.5 * u)
            e.index_add_(0, j, 0.5 * u)
        return F, e, W


def _spread3(v):
    v = v & 0x3FF
    for s, m in ((16, 0xFF0000FF), (8, 0x0300F00F), (4, 0x030C30C3), (2, 0x09249249)):
        v = (v ^ (v << s)) & m
    return v


def _morton_order(systems):
    """Rows of the concatenated systems after the first build's sort."""
    out, base = [], 0
    for s in systems:
        q = np.clip(np.floor(s["pos"] * (1024.0 / s["L"])), 0, 1023).astype(np.int64)
        code = _spread3(q[:, 0]) | (_spread3(q[:, 1]) << 1) | (_spread3(q[:, 2]) << 2)
        out.append(base + np.argsort(code, kind="stable"))
        base += s["pos"].shape[0]
    return np.concatenate(out)


def _four(x, w=None):
    z = torch.zeros((x.shape[0], 4), dtype=torch.float64, device=x.device)
    z[:, :3] = x
    if w is not None:
        z[:, 3] = w
    return z


def _fold(x, L):
    x = torch.where(x >= L, x - L, torch.where(x < 0, x + L, x))
    return torch.where(x >= L, x - L, x)


def exact(case, seed):
    seed = 7 + 100003 * (seed % 20000)
    dev = _device()
    t64 = lambda a: torch.as_tensor(np.asarray(a, dtype=np.float64), device=dev)  # noqa: E731
    if case["kind"] in ("exchange", "reselect"):
        sysd, gpos, gtag, _, _, _ = _subdomain(case, seed)
        n, cap = sysd["pos"].shape[0], sysd["n_cap"]
        allr = dict(sysd, pos=np.concatenate([sysd["pos"], gpos]))
        x = t64(allr["pos"])
        F, _, _ = _Model([allr], ["lj"], dev, 0.0)(x, None, 0)
        force, pos = torch.zeros((cap, 4), dtype=torch.float64, device=dev), torch.zeros(
            (cap, 4), dtype=torch.float64, device=dev)
        force[:n, :3] = F[:n]
        pos[:x.shape[0], :3] = x
        return dict(force=force, pos=pos, tag=None, send=None, counts=None, offsets=None)
    if case["kind"] == "batch":
        ens = _ensemble(case, seed)
        fluids, systems = [f for f, _ in ens], [s for _, s in ens]
    else:
        fluids, systems = [case["fluid"]], [_system(case["fluid"], case["n"], seed)]
    order = _morton_order(systems)
    x = t64(np.concatenate([s["pos"] for s in systems]))
    v = t64(np.concatenate([s["vel"] for s in systems]))
    n = x.shape[0]
    at = torch.as_tensor(order, device=dev)
    if case["kind"] == "evaluate":
        F, e, W = _Model(systems, fluids, dev, 0.0)(x, v, 0)
        ke = 0.5 * float((v * v).sum())
        thermo = np.array([[ke, float(e.sum()), W, 2.0 * ke / (3.0 * n - 3.0)]])
        return dict(force=_four(F, e)[at], pos=_four(x)[at], tag=None, thermo=thermo)
    model = _Model(systems, fluids, dev, 0.4 if fluids[0] != "dpd" else 0.5)
    L, dt = model.pairs.L, _params(fluids[0], True).dt
    nvt = fluids[0] == "weak"
    xi, steps, log, rows = 0.0, case["steps"], case.get("log", 0), []
    g = 3.0 * n - 3.0

    def note(s, e, W):
        if log and (s % log == 0 or s == steps):
            ke = 0.5 * float((v * v).sum())
            rows.append([[float(s), ke, float(e.sum()), W, 2.0 * ke / g]])

    F, e, W = model(x, v, 0)
    note(0, e, W)
    for s in range(steps):
        v = v + 0.5 * dt * (F - xi * v)
        x = _fold(x + dt * v, L)
        if nvt:
            xi = xi + dt / 0.25 * (float((v * v).sum()) / g / 1.2 - 1.0)
        F, e, W = model(x, v, s + 1)
        v = (v + 0.5 * dt * F) / (1.0 + 0.5 * dt * xi)
        note(s + 1, e, W)
    # a step's force array carries the energies when the step is logged
    out = dict(pos=_four(x)[at], vel=_four(v)[at], force=_four(F, e if log else None)[at], tag=None)
    if log:
        out["log"] = np.array(rows)
    return out
