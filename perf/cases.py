"""Timed cases: the work a user has this library do, through its public entry points.

A case is a dict of plain values. `kind` names the call sequence:

  point    a new structure (or batch of structures): list build, then energies, forces and
           uncertainties of every atom: a request of a serving lane (in the lane's large
           state) or one active-learning candidate. With virial, the per-cell virial as well
  eval     energies, forces and uncertainties at given positions on a list that is kept: an
           external integrator, a relaxation
  md       ten velocity-Verlet steps (one interval between two list builds)
  nvt      ten Nose-Hoover steps with the production-run analysis at the end of the interval
  grad     forward and backward of the energies as a torch module
  screen   uncertainties alone (no energies, no forces) of new structures
  desc     descriptors and their norms written out for new structures

and `geom` the structures: `gas` an H2 gas column over a Pt(111) slab (nx, ny, layers,
height, tiled tx by ty), `slabs` adsorbed Pt(111) slabs (count of them, log-uniform sizes
between lo and hi atoms), `cells` small 6x6x4 slabs with 4 to 32 H2 each, `tiny` the 80-atom
cell. Every atom gets a seeded jitter, so another seed is another input. The model is the
random positive semi-definite one with 544 components.

Per-cell energies come out of the library as FP64 sums of FP32 per-atom energies, and a
module's gradients as FP32 forces in the dtype of the positions: both are returned as the
FP32 values whose accuracy they have.
"""
import math

import numpy as np
import torch

from paper_2204_12573_amd import autograd, binding, engine
from paper_2204_12573_amd import structures as S

R_CUT, N_RAD, N_DESC = 4.5, 8, 544
KAPPA, KB = 9.648533212e-3, 8.617333262e-5
PRECISION = {"fp32": binding.FP32, "bf16": binding.BF16_SPLIT, "fp8": binding.FP8_SPLIT,
             "bf16x6": binding.BF16X6_SPLIT, "bf16x6_var32": binding.BF16X6_SPLIT | binding.VAR_FP32}
# Trajectories: production runs' 0.1 fs steps. A cold start, because the random model binds
# nothing: the structure then stays the case's own over the few hundred fs that repeated
# passes on one state add up to.
DT, SKIN, EVERY, T_MD, TAU = 0.1, 0.2, 10, 50.0, 10.0


def listed():
    return [
        # one small candidate structure, alone: launches and latency
        {"name": "point_80", "kind": "point", "geom": "tiny", "prec": "fp32"},
        # a small slab's trajectory: latency again, without list builds in most steps
        {"name": "md_1k", "kind": "md", "geom": "slabs", "count": 1, "lo": 1217, "hi": 1217, "prec": "fp32"},
        # eight cells of a training batch, energies and their gradient
        {"name": "grad_8", "kind": "grad", "geom": "cells", "count": 8, "prec": "fp32"},
        # the differentiation batch
        {"name": "grad_256", "kind": "grad", "geom": "cells", "count": 256, "prec": "fp32"},
        # one request of ordinary size with the stress
        {"name": "point_7k_virial", "kind": "point", "geom": "slabs", "count": 1, "lo": 7893, "hi": 7893,
         "virial": True, "prec": "fp32"},
        # a serving lane's batch under load, in the form the server is run with
        {"name": "serve_batch_bf16", "kind": "point", "geom": "slabs", "count": 24, "lo": 100, "hi": 50000,
         "lane": True, "prec": "bf16"},
        # candidates screened by uncertainty alone
        {"name": "screen_300", "kind": "screen", "geom": "cells", "count": 300, "prec": "fp32"},
        # descriptors written out, to choose a sparse set
        {"name": "desc_20k", "kind": "desc", "geom": "slabs", "count": 3, "lo": 3001, "hi": 15013, "prec": "fp32"},
        # a production run of ordinary size: thermostat, coordination, reaction events, monitor
        {"name": "nvt_50k", "kind": "nvt", "geom": "slabs", "count": 1, "lo": 49952, "hi": 49952, "prec": "fp32"},
        # trajectory with the FP64 variance and the three-way energy pass
        {"name": "md_200k_bf16x6", "kind": "md", "geom": "gas", "nx": 25, "ny": 20, "layers": 24, "height": 1142.2,
         "tx": 2, "ty": 2, "prec": "bf16x6"},
        # the headline trajectory: about a million atoms, energies, forces and uncertainties
        {"name": "md_1m", "kind": "md", "geom": "gas", "nx": 25, "ny": 20, "layers": 24, "height": 1142.2,
         "tx": 4, "ty": 5, "prec": "fp32"},
        # the largest: one evaluation of four million atoms
        {"name": "eval_4m", "kind": "eval", "geom": "gas", "nx": 25, "ny": 20, "layers": 24, "height": 1142.2,
         "tx": 8, "ty": 10, "prec": "fp32"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["point", "point", "eval", "md", "md", "nvt", "grad", "screen", "desc"])
    case = {"kind": kind, "prec": rng.choice(["fp32", "fp32", "bf16", "bf16x6", "bf16x6_var32", "fp8"])}
    most = {"point": 400000, "eval": 2000000, "md": 900000, "nvt": 400000, "grad": 60000, "screen": 200000,
            "desc": 60000}[kind]
    if kind in ("eval", "md") and rng.random() < 0.6:
        # an H2 column over a slab: thin and thick slabs, dilute to slab-only heights
        nx, ny = rng.randint(5, 24), 2 * rng.randint(3, 12)
        layers, height = rng.randint(3, 24), round(rng.uniform(15.0, 1100.0), 1)
        n = nx * ny * layers + 2 * int(S.GAS_DENSITY * nx * ny * S.A_NN * S.ROW * height)
        tx = max(1, min(12, int(math.sqrt(_log_int(rng, 2000, most) / n))))
        ty = max(1, min(tx + rng.randint(0, 2), int(most / n / tx)))
        case.update(geom="gas", nx=nx, ny=ny, layers=layers, height=height, tx=tx, ty=ty)
    elif kind in ("grad", "screen") or (kind == "point" and rng.random() < 0.3):
        case.update(geom="cells", count=_log_int(rng, 1, most // 180))
    elif kind in ("point", "desc"):
        hi = _log_int(rng, 120, min(most, 50000))
        case.update(geom="slabs", count=_log_int(rng, 1, max(1, min(64, most // hi))), lo=max(60, hi // 20), hi=hi)
    else:
        n = _log_int(rng, 100, most)
        case.update(geom="slabs", count=1, lo=n, hi=n)
    if kind == "point":
        case["virial"] = rng.random() < 0.3
        case["lane"] = rng.random() < 0.5
    return case


# ---- inputs ----

def _slab_sizes(case):
    k = case["count"]
    return [int(round(case["lo"] * (case["hi"] / case["lo"]) ** ((i + 0.5) / k))) for i in range(k)]


def _inputs(case, seed):
    """Positions [N, 3], species, offsets, boxes of the case, from the seed alone."""
    rng = np.random.default_rng(seed)
    if case["geom"] == "tiny":
        b = S.concat([S.config_tiny(seed=seed)])
    elif case["geom"] == "cells":
        b = S.concat([S.h2_over_pt111(6, 6, 4, vacuum=15.0, n_mol=4 + 11 * i % 29, jitter=0.1,
                                      seed=seed % 100003 * 1009 + i) for i in range(case["count"])])
    elif case["geom"] == "slabs":
        # the sizes are the case's own, whatever the seed: evenly spread over the logarithm
        b = S.concat([S.adsorbed_slab(n, 0.1 + 0.37 * i % 0.9, int(rng.integers(1 << 30)))
                      for i, n in enumerate(_slab_sizes(case))])
    else:
        st = S.h2_over_pt111(case["nx"], case["ny"], case["layers"], gas_height=case["height"], jitter=0.0, seed=seed)
        st = S.tiled(st, case["tx"], case["ty"])
        pos = st.pos + rng.standard_normal(st.pos.shape, dtype=np.float32) * 0.05
        b = S.Batch(pos - st.box * np.floor(pos / st.box), st.species, np.array([0, st.n], np.int32), st.box[None])
    return b


def _velocities(case, b, seed):
    m = S.MASS[b.species]
    v = np.random.default_rng(seed + 1).standard_normal((b.n, 3)) * np.sqrt(KB * T_MD * KAPPA / m)[:, None]
    if case["geom"] == "gas":             # the two atoms of a gas molecule travel together
        h = np.nonzero(b.species == S.H)[0]
        v[h[0::2]] = v[h[1::2]] = (v[h[0::2]] + v[h[1::2]]) / math.sqrt(2.0)
    return v - (m[:, None] * v).sum(0) / m.sum()


def prepare(case, seed):
    b = _inputs(case, seed)
    beta, sigma = S.random_model(N_DESC)
    model = engine.Model(beta, sigma, precision=PRECISION[case["prec"]])
    pos, species = engine.to_device(b.pos, b.species)
    pairs = (16 if case["geom"] == "gas" and case["height"] > 200 else 48) * b.n + 4096
    s = {"case": case, "kind": case["kind"], "offsets": b.offsets, "boxes": b.boxes, "pos": pos, "species": species}
    if s["kind"] == "grad":
        s["module"] = autograd.FlareEnergy(model, species, b.offsets, b.boxes)
        s["pos"] = pos.requires_grad_(True)
        w = np.random.default_rng(seed + 2).standard_normal(len(b.boxes))
        s["weight"] = torch.from_numpy(w).cuda()
        return s
    if case.get("lane"):                  # a serving lane's state is larger than most batches
        ev = engine.Evaluator(model, max_atoms=400000, max_pairs=22 * 400000)
    else:
        ev = engine.Evaluator(model, max_atoms=b.n, max_pairs=pairs)
    s["ev"] = ev
    if s["kind"] in ("md", "nvt"):
        vel = torch.from_numpy(np.ascontiguousarray(_velocities(case, b, seed).T)).cuda()
        args = (ev, pos, vel, species, b.offsets, b.boxes)
        if s["kind"] == "md":
            s["md"] = engine.MD(*args, dt=DT, skin=SKIN, rebuild=EVERY)
        else:
            s["md"] = engine.NVT(*args, t_target=T_MD, tau=TAU, dt=DT, skin=SKIN, rebuild=EVERY)
            s["run"] = engine.Production(s["md"], every=EVERY)
    elif s["kind"] == "eval":
        # positions a little away from those of the list build
        ev.neighbors(pos, species, b.offsets, b.boxes, SKIN)
        step = np.random.default_rng(seed + 3).uniform(-0.05, 0.05, (3, b.n))
        s["pos"] = pos + torch.from_numpy(step).cuda()
        s["out"] = ev.compute(s["pos"])
    else:
        s["out"] = {}
    return s


def run(s):
    kind = s["kind"]
    if kind == "grad":
        energy = s["module"](s["pos"])
        (g,) = torch.autograd.grad(energy, s["pos"], s["weight"])
        return {"E": energy.detach().float(), "grad": g.float()}
    ev, pos = s["ev"], s["pos"]
    if kind in ("md", "nvt"):
        md, work = s["md"], s.get("run", s["md"])
        for _ in range(EVERY):
            out = work.step()
        got = {"pos": md.pos, "vel": md.vel, "e": out["e"], "f": out["f"], "var": out["var"], "sigma": out["sigma"],
               "E": out["E"].float()}
        if kind == "nvt":
            got.update(thermo=md.thermo, coord=work.coord, events=work.events, sigma_max=work.sigma_max,
                       over=work.over)
        return got
    if kind != "eval":
        ev.neighbors(pos, s["species"], s["offsets"], s["boxes"], 0.0)
    if kind == "desc":
        d, norm = ev.descriptors(pos, want_d=True, want_norm=True)
        return {"d": d, "norm": norm}
    if kind == "screen":
        ev.descriptors(pos)
        out = s["out"] = ev.variance(s["out"])
        return dict(out)
    out = s["out"] = ev.compute(pos, out=s["out"])
    got = {"e": out["e"], "f": out["f"], "var": out["var"], "sigma": out["sigma"], "E": out["E"].float()}
    if s["case"].get("virial"):
        got["virial"] = ev.virial().float()
    return got


# ---- what a pass cannot do without ----

def work(case):
    """Inputs once, outputs once, and the arithmetic of the method: per listed pair inside the
    cutoff the density (320 flop) and the adjoint term (830); per row the quadratic forms of
    its width (2 n^2 for the energy and its gradient, n^2 through the variance's triangular
    factor) and the contractions around them. The atoms that see both species are estimated
    from the surface area."""
    if case["geom"] == "tiny":
        n, sites, pairs, mixed = 80, 16, 14 * 64, 40
    elif case["geom"] == "cells":
        k = case["count"]
        n, sites, pairs, mixed = 180 * k, 36 * k, 2400 * k, 90 * k
    elif case["geom"] == "slabs":
        n = sum(_slab_sizes(case))
        sites = n / 4.5
        pairs, mixed = 15 * n, int(2.4 * sites)
    else:
        cells = case["tx"] * case["ty"]
        sites = case["nx"] * case["ny"] * cells
        h = 2 * S.GAS_DENSITY * sites * S.A_NN * S.ROW * case["height"]
        n = int(sites * case["layers"] + h)
        pairs, mixed = int(18 * sites * case["layers"] + 2 * h), int(1.35 * sites)
    single = max(0, n - mixed)
    want_e, want_v = case["kind"] not in ("screen", "desc"), case["kind"] not in ("grad", "desc")
    form = (2 if want_e else 0) + (1 if want_v else 0)
    flops = pairs * (320 + (830 if want_e else 0)) + single * (form * 144 * 144 + 1440) \
        + mixed * (form * N_DESC * N_DESC + 5440)
    if want_e:
        flops += single * 3000 + mixed * 12000
    io = {"point": 28 + 24, "eval": 24 + 24, "md": 124 + 24, "nvt": 124 + 24, "grad": 28 + 24, "screen": 28 + 8,
          "desc": 28 + 4 * N_DESC + 4}[case["kind"]]
    weights = 4 * form * N_DESC * N_DESC
    steps = EVERY if case["kind"] in ("md", "nvt") else 1
    return {"bytes": steps * (n * io + weights), "flops": steps * flops}


# ---- the same in 64 bits, from the definitions ----

def _pairs(pos, cell, boxes, r_list):
    """Directed pairs (i, j, image shift) with |x_j - x_i + s L| < r_list, all cells at once."""
    dev, n = pos.device, len(pos)
    nb = torch.clamp(torch.floor(boxes / r_list), 1, 512)
    reach = torch.ceil(r_list / (boxes / nb)).max(0).values.long().tolist()
    size = nb.prod(1).long()
    base = torch.cumsum(size, 0) - size
    nbl = nb.long()[cell]
    at = torch.minimum((pos / (boxes / nb)[cell]).long(), nbl - 1)

    def index(b):
        return base[cell] + (b[:, 2] * nbl[:, 1] + b[:, 1]) * nbl[:, 0] + b[:, 0]

    order = torch.argsort(index(at))
    count = torch.bincount(index(at), minlength=int(size.sum()))
    start = torch.cumsum(count, 0) - count
    every, found = torch.arange(n, device=dev), []
    for oz in range(-reach[2], reach[2] + 1):
        for oy in range(-reach[1], reach[1] + 1):
            for ox in range(-reach[0], reach[0] + 1):
                to = at + torch.tensor([ox, oy, oz], device=dev)
                shift = torch.div(to, nbl, rounding_mode="floor")
                b = index(to - shift * nbl)
                c = count[b]
                i = torch.repeat_interleave(every, c)
                first = torch.cumsum(c, 0) - c
                j = order[start[b][i] + torch.arange(len(i), device=dev) - first[i]]
                d = pos[j] - pos[i] + shift[i] * boxes[cell[i]]
                keep = ((d * d).sum(1) < r_list * r_list) & ((i != j) | (shift[i] != 0).any(1))
                found.append((i[keep], j[keep], (shift[i[keep]] * boxes[cell[i[keep]]])))
    i, j, s = (torch.cat(x) for x in zip(*found))
    by = torch.argsort(i, stable=True)
    return i[by], j[by], s[by]


def _harmonics(u):
    x, y, z = u.unbind(-1)
    xx, yy, zz, q = x * x, y * y, z * z, math.sqrt(1.0 / math.pi)
    r = [0.5 * q + 0 * x,
         *(math.sqrt(0.75) * q * t for t in (y, z, x)),
         *(math.sqrt(15.0) / 2 * q * t for t in (x * y, y * z, (3 * zz - 1) / math.sqrt(12.0), x * z, (xx - yy) / 2)),
         math.sqrt(35.0 / 32) * q * y * (3 * xx - yy), math.sqrt(105.0) / 2 * q * x * y * z,
         math.sqrt(21.0 / 32) * q * y * (5 * zz - 1), math.sqrt(7.0) / 4 * q * z * (5 * zz - 3),
         math.sqrt(21.0 / 32) * q * x * (5 * zz - 1), math.sqrt(105.0) / 4 * q * z * (xx - yy),
         math.sqrt(35.0 / 32) * q * x * (xx - 3 * yy)]
    return torch.stack(r, -1)


class _Exact:
    """Energies, variances, forces and virials in FP64, the gradient by torch's autograd over
    chunks of atoms."""

    def __init__(self, b):
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        off = torch.from_numpy(np.asarray(b.offsets, np.int64)).to(dev)
        self.n, self.cells = b.n, len(b.boxes)
        self.sizes = (off[1:] - off[:-1]).tolist()
        self.cell = torch.repeat_interleave(torch.arange(self.cells, device=dev), off[1:] - off[:-1])
        self.boxes = torch.from_numpy(np.asarray(b.boxes, np.float64)).to(dev)
        self.pos = torch.from_numpy(np.asarray(b.pos, np.float64)).to(dev)
        self.sp = torch.from_numpy(np.asarray(b.species, np.int64)).to(dev)
        beta, sigma = S.random_model(N_DESC)
        self.beta, self.sigma = torch.from_numpy(beta).to(dev), torch.from_numpy(sigma).to(dev)
        packed = []                       # channel pairs a <= b, by species pair, row-major
        for s1, s2 in ((0, 0), (0, 1), (1, 1)):
            for p in range(N_RAD):
                for q in range(p if s1 == s2 else 0, N_RAD):
                    packed.append((s1 * N_RAD + p) * 2 * N_RAD + s2 * N_RAD + q)
        self.packed = torch.tensor(packed, device=dev)

    def list(self, skin):
        wrapped = self.pos - self.boxes[self.cell] * torch.floor(self.pos / self.boxes[self.cell])
        i, j, s = _pairs(wrapped, self.cell, self.boxes, R_CUT + skin)
        base = self.pos - wrapped
        self.i, self.j, self.s = i, j, s - base[j] + base[i]

    def per_cell(self, v):
        return torch.stack([t.sum(0) for t in torch.split(v, self.sizes)])

    def evaluate(self, want_f=True, want_d=False, chunk=32768):
        dev, n = self.pos.device, self.n
        out = {"e": torch.zeros(n, dtype=torch.float64, device=dev), "var": torch.zeros(n, dtype=torch.float64, device=dev),
               "norm": torch.zeros(n, dtype=torch.float64, device=dev)}
        f = torch.zeros((n, 3), dtype=torch.float64, device=dev)
        virial = torch.zeros((n, 9), dtype=torch.float64, device=dev)
        d_all = []
        first = torch.searchsorted(self.i, torch.arange(0, n + chunk, chunk, device=dev)).tolist()
        for k, lo in enumerate(range(0, n, chunk)):
            hi = min(n, lo + chunk)
            i, j, s = (t[first[k]:first[k + 1]] for t in (self.i, self.j, self.s))
            delta = self.pos[j] - self.pos[i] + s
            keep = (delta * delta).sum(1) < R_CUT * R_CUT
            i, j, delta = i[keep], j[keep], delta[keep].requires_grad_(want_f)
            r = delta.square().sum(1).sqrt()
            x = 2.0 * r / R_CUT - 1.0
            t = [torch.ones_like(x), x]
            while len(t) < N_RAD:
                t.append(2.0 * x * t[-1] - t[-2])
            radial = torch.stack(t, 1) * ((R_CUT - r) ** 2)[:, None]
            # the pairs of an atom side by side, so that the densities are a sum per atom
            count = torch.bincount(i - lo, minlength=hi - lo)
            most = max(1, int(count.max()))
            slot = (i - lo) * most + torch.arange(len(i), device=dev) - (torch.cumsum(count, 0) - count)[i - lo]
            y = torch.zeros(((hi - lo) * most, 16), dtype=torch.float64, device=dev)
            y = y.index_copy(0, slot, _harmonics(delta / r[:, None])).reshape(hi - lo, most, 16)
            by = torch.zeros(((hi - lo) * most, 2, N_RAD), dtype=torch.float64, device=dev)
            by = by.index_copy(0, slot, torch.nn.functional.one_hot(self.sp[j], 2)[:, :, None] * radial[:, None, :])
            c = (by.reshape(hi - lo, most, 2 * N_RAD, 1) * y[:, :, None, :]).sum(1)
            parts = [c[:, :, m0:m1] for m0, m1 in ((0, 1), (1, 4), (4, 9), (9, 16))]
            dt = torch.stack([(q[:, :, None] * q[:, None, :]).sum(-1).reshape(hi - lo, -1)
                              .index_select(1, self.packed) for q in parts], -1).reshape(hi - lo, N_DESC)
            norm2 = dt.square().sum(1)
            none = norm2 == 0
            norm = torch.where(none, torch.ones_like(norm2), norm2).sqrt()
            d = dt / norm[:, None]
            heavy, flat = self.sp[lo:hi] == 1, d.detach()
            e = torch.where(heavy, ((d @ self.beta[1]) * d).sum(1), ((d @ self.beta[0]) * d).sum(1))
            out["var"][lo:hi] = torch.where(heavy, ((flat @ self.sigma[1]) * flat).sum(1),
                                            ((flat @ self.sigma[0]) * flat).sum(1))
            if want_f and len(i):
                (h,) = torch.autograd.grad(e.sum(), delta)
                f.index_add_(0, i, h)
                f.index_add_(0, j, -h)
                virial.index_add_(0, i, -(delta.detach()[:, :, None] * h[:, None, :]).reshape(-1, 9))
            out["e"][lo:hi] = e.detach()
            out["norm"][lo:hi] = torch.where(none, 0.0, norm.detach())
            if want_d:
                d_all.append(d.detach())
        out["sigma"] = out["var"].clamp(min=0).sqrt()
        out["f"], out["virial"], out["E"] = f, self.per_cell(virial).reshape(-1, 3, 3), self.per_cell(out["e"])
        if want_d:
            out["d"] = torch.cat(d_all)
        return out


def exact(case, seed):
    if case["kind"] in ("md", "nvt") and work(case)["flops"] > 1.2e12:
        return None                       # ten steps in 64 bits take too long
    b = _inputs(case, seed)
    x = _Exact(b)
    kind = case["kind"]
    if kind in ("md", "nvt"):
        return _exact_md(x, b, case, seed)
    x.list(SKIN if kind == "eval" else 0.0)
    if kind == "eval":
        step = np.random.default_rng(seed + 3).uniform(-0.05, 0.05, (3, b.n))
        x.pos = x.pos + torch.from_numpy(step.T).to(x.pos.device)
    o = x.evaluate(want_f=kind not in ("desc", "screen"), want_d=kind == "desc")
    if kind == "grad":
        w = torch.from_numpy(np.random.default_rng(seed + 2).standard_normal(x.cells)).to(x.pos.device)
        return {"E": o["E"], "grad": -(w[x.cell][:, None] * o["f"]).T.contiguous()}
    if kind == "desc":
        return {"d": o["d"], "norm": o["norm"]}
    if kind == "screen":
        top = torch.stack([t.max() for t in torch.split(o["sigma"], x.sizes)])
        return {"var": o["var"], "sigma": o["sigma"], "sigma_max": top}
    got = {"e": o["e"], "f": o["f"].T.contiguous(), "var": o["var"], "sigma": o["sigma"], "E": o["E"]}
    if case.get("virial"):
        got["virial"] = o["virial"]
    return got


def _exact_md(x, b, case, seed):
    kind = case["kind"]
    v = torch.from_numpy(_velocities(case, b, seed)).to(x.pos.device)
    m = torch.from_numpy(engine.MASSES).to(x.pos.device)[x.sp][:, None]
    x.list(SKIN)
    o = x.evaluate()
    nf = max(3 * b.n - 3, 1)
    zeta, eta, top = 0.0, 0.0, None
    kin = (m * v * v).sum() / (2 * KAPPA)

    def friction(k):
        return 0.5 * DT * (2.0 * k / (nf * KB * T_MD) - 1.0) / TAU ** 2

    for step in range(EVERY):
        if kind == "nvt":
            zeta = zeta + friction(kin)
            v = v * torch.exp(-zeta * DT / 2)
            eta = eta + zeta * DT / 2
        v = v + 0.5 * DT * KAPPA * o["f"] / m
        x.pos = x.pos + DT * v
        if step == EVERY - 1:
            x.list(SKIN)
        o = x.evaluate()
        v = v + 0.5 * DT * KAPPA * o["f"] / m
        if kind == "nvt":
            v = v * torch.exp(-zeta * DT / 2)
            eta = eta + zeta * DT / 2
            kin = (m * v * v).sum() / (2 * KAPPA)
            zeta = zeta + friction(kin)
    got = {"pos": x.pos.T.contiguous(), "vel": v.T.contiguous(), "e": o["e"], "f": o["f"].T.contiguous(),
           "var": o["var"], "sigma": o["sigma"], "E": o["E"]}
    if kind == "nvt":
        top = o["sigma"].max().reshape(1)
        got.update(thermo=torch.stack([zeta, eta, kin])[None], coord=None, events=None, sigma_max=top, over=None)
    return got
