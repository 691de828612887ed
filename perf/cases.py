"""Workloads of the framework through its public entry points.

Every case is a dict of plain values.  ``listed()`` names the standing ones,
``draw(rng)`` gives one more of the same ranges, ``prepare(case, seed)`` makes
what a planning program holds before the call (inputs, engine, loaded
geometry), ``run(state)`` is one pass through the public entry points and
returns its outputs whole, ``work(case)`` the bytes and operations the pass
cannot do without, ``exact(case, seed)`` the outputs in 64 bits where such
values exist (Monte Carlo transport has none: its outputs are held to be the
same numbers for the same seed).

Kinds
  dose       dense dose of one field (``Engine.run_dose``)
  im         influence matrices of all fields and scenarios (``Engine.run_csr``)
  optimize   robust spot weights from influence matrices (``Engine.optimize``)
  cells      influence matrices merged into coarser cells (``vpmc_csr_cells``)
  surrogate  training epochs of the aperture network and a forward pass on
             held-out entries (``vpmc_surrogate_train`` / ``_forward``)
"""
import copy
import functools
import math
import weakref

import numpy as np
import torch

from paper_2307_01416_amd import inputs as I
from paper_2307_01416_amd import vpmc as V

HEAD, HEAD_MM = I.HEAD_SHAPE, I.HEAD_SPACING
FULL, STRAIGHT = I.PHYS_ALL, 0


# ------------------------------------------------------------------- cases
def _water_dose(opening, rs, vps, shape, mm, batches=16, physics=FULL, energy=100.0):
    """Water phantom; opening 0: one open pencil beam of the given energy."""
    return {"kind": "dose", "geom": "water", "opening_mm": float(opening), "rs": bool(rs), "vps": int(vps),
            "nx": shape[0], "ny": shape[1], "nz": shape[2], "mm": float(mm), "batches": batches,
            "physics": physics, "let": False, "scenarios": 1, "energy": float(energy)}


def _head_dose(cc, gantry, vps, batches=16, physics=FULL, let=False, scenarios=1):
    """Head CT, one field behind aperture and range shifter; vps per spot."""
    return {"kind": "dose", "geom": "head", "target_cc": cc, "gantry": float(gantry), "vps": int(vps),
            "batches": batches, "physics": physics, "let": let, "scenarios": scenarios}


def _water_im(opening, rs, vps, shape, mm):
    return {"kind": "im", "geom": "water", "opening_mm": float(opening), "rs": bool(rs), "vps": int(vps),
            "nx": shape[0], "ny": shape[1], "nz": shape[2], "mm": float(mm), "physics": FULL, "scenarios": 1,
            "energy": 0.0}


def _head_im(cc, fields, vps, scenarios=13):
    return {"kind": "im", "geom": "head", "target_cc": cc, "fields": fields, "vps": int(vps), "physics": FULL,
            "scenarios": scenarios}


def _rows(kind, shape, spots, scen, **kw):
    """Pencil-beam-like rows on a grid (optimiser, cell merge)."""
    return {"kind": kind, "nx": shape[0], "ny": shape[1], "nz": shape[2], "spots": int(spots), "scen": int(scen), **kw}


def listed():
    return [
        # the smallest plan check: one 100 MeV pencil beam into 2 mm water
        # with its batch uncertainty, called interactively
        {"name": "dose_water_pencil", **_water_dose(0, False, 100_000, (50, 50, 100), 2.0)},
        # the paper's energy-layer validation: 20 mm opening behind the range
        # shifter, 1 mm water, 1e7 particles, uncertainty from 16 batches
        {"name": "dose_water_layer", **_water_dose(20, True, 10_000_000, (200, 200, 300), 1.0)},
        # plan dose of one field of the 8 cc head case with uncertainty
        {"name": "dose_head_field", **_head_dose(8.0, 180.0, 10_000)},
        # robustness evaluation with LET: one field under three scenarios,
        # no uncertainty
        {"name": "dose_head_let", **_head_dose(8.0, 90.0, 3_000, batches=0, let=True, scenarios=3)},
        # deterministic (straight CSDA) check of a small-target field
        {"name": "dose_head_straight", **_head_dose(0.4, 270.0, 4_000, batches=0, physics=STRAIGHT)},
        # influence matrix of one energy layer in water, nominal only
        {"name": "im_water_layer", **_water_im(10, True, 20_000, (200, 200, 300), 1.0)},
        # small brain target: 3 fields, 13 robust scenarios
        {"name": "im_head_small_target", **_head_im(0.4, 3, 5_000)},
        # 8 cc target: 2 fields, 13 robust scenarios
        {"name": "im_head_8cc", **_head_im(8.0, 2, 8_000)},
        # optimiser on the shape of its tests: everything is latency
        {"name": "optimize_small", **_rows("optimize", (40, 36, 20), 48, 3, iters=80, reuse=False)},
        # optimiser on the head grid, 13 scenarios
        {"name": "optimize_head", **_rows("optimize", HEAD, 600, 13, iters=80, reuse=False)},
        # dynamic voxel spacing of the head matrices
        {"name": "cells_head", **_rows("cells", HEAD, 600, 13)},
        # training of the aperture network: forward and backward
        {"name": "surrogate_train", "kind": "surrogate", "n": 131_072, "batch": 4096, "epochs": 2, "held": 65_537},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["dose_water", "dose_water", "dose_head", "dose_head", "im_water", "im_head", "im_head",
                       "optimize", "optimize", "cells", "surrogate"])
    if kind == "dose_water":
        mm = rng.choice([1.0, 2.0])
        shape = (rng.randint(45, 201), rng.randint(45, 201), rng.randint(100, 300) if mm == 1.0 else rng.randint(60, 150))
        opening = rng.choice([0, 10, 20, 30, 40])
        return _water_dose(opening, opening and rng.random() < 0.5, _log(rng, 20_000, 8_000_000), shape, mm,
                           batches=rng.choice([0, 10, 16, 20]), physics=rng.choice([FULL, FULL, FULL, STRAIGHT]),
                           energy=round(rng.uniform(71.3, 200.0), 1))
    if kind == "dose_head":
        return _head_dose(rng.choice([0.4, 8.0]), rng.choice([0.0, 90.0, 135.0, 180.0, 270.0]), _log(rng, 300, 9_000),
                          batches=rng.choice([0, 16, 16, 10]), physics=rng.choice([FULL, FULL, FULL, STRAIGHT]),
                          let=rng.random() < 0.25, scenarios=rng.choice([1, 1, 2]))
    if kind == "im_water":
        return _water_im(rng.choice([10, 20, 30, 40]), rng.random() < 0.5, _log(rng, 500, 20_000),
                         (rng.randint(90, 200), rng.randint(90, 200), rng.randint(180, 300)), 1.0)
    if kind == "im_head":
        cc = rng.choice([0.4, 8.0])
        return _head_im(cc, rng.choice([1, 2, 3]) if cc == 0.4 else 1, _log(rng, 500, 5_000 if cc == 0.4 else 2_500),
                        scenarios=rng.choice([1, 5, 13]))
    if kind == "optimize":
        shape = (rng.randint(40, 256), rng.randint(36, 256), rng.randint(20, 160))
        return _rows("optimize", shape, _log(rng, 30, 500), rng.choice([1, 3, 13]), iters=rng.choice([40, 80, 150]),
                     reuse=rng.random() < 0.4)
    if kind == "cells":
        return _rows("cells", (rng.randint(40, 256), rng.randint(36, 256), rng.randint(20, 160)), _log(rng, 30, 500),
                     rng.choice([1, 3, 13]))
    return {"kind": "surrogate", "n": _log(rng, 8_192, 131_072), "batch": rng.choice([512, 2048, 4096, 5000]),
            "epochs": rng.choice([1, 2]), "held": _log(rng, 1_000, 65_536)}


# --------------------------------------------------------------- transport
@functools.lru_cache(maxsize=1)
def _head_ct():
    return I.head_ct(0)


@functools.lru_cache(maxsize=8)
def _head_plan(cc, gantries):
    """The plan on the head CT: fields with their apertures and spot layers."""
    return I.config3(cc, 1000, geometry=_head_ct(), gantries=gantries)


_GEOM, _ENGINES = weakref.WeakValueDictionary(), weakref.WeakValueDictionary()


def _water(c):
    key = (c["nx"], c["ny"], c["nz"], c["mm"])
    g = _GEOM.get(key)
    if g is None:
        _GEOM[key] = g = I.water_geometry(key[:3], (c["mm"],) * 3)
    return g


def _engine_of(geometry):
    """The engine that a planning program keeps for one patient: influence
    matrices of all its plans run on it."""
    e = _ENGINES.get(id(geometry))
    if e is None:
        _ENGINES[id(geometry)] = e = V.Engine(0)
    return e


def _scenarios(n, rng):
    """Nominal first; then scenarios of the robust set in a seeded order."""
    s = I.scenarios_13()
    return s if n == 13 else s[:1] + [s[1 + int(i)] for i in rng.permutation(12)[: n - 1]]


def _case(c, seed):
    """The plan of a transport case; the seed gives the delivered spot
    positions (0.2 mm), weights, history counts and the particles' streams."""
    rng = np.random.default_rng(seed)
    im = c["kind"] == "im"
    if c["geom"] == "head":
        gantries = (c["gantry"],) if not im else {1: (180.0,), 2: (180.0, 270.0), 3: (90.0, 180.0, 270.0)}[c["fields"]]
        base = _head_plan(c["target_cc"], gantries)
        per_spot = c["vps"]
    elif c["opening_mm"] > 0:
        base = I.config2(c["opening_mm"], c["rs"], shape=(c["nx"], c["ny"], c["nz"]), spacing=(c["mm"],) * 3)
        base.geometry = _water(c)
        per_spot = c["vps"] if im else max(1, c["vps"] // len(base.fields[0].spots))
    else:
        g = _water(c)
        iso = (0.5 * c["nx"] * c["mm"], 0.5 * c["ny"] * c["mm"], 0.0)
        spots = I.make_spots([(0.0, 0.0)], c["energy"], I.spot_sigma_mm(c["energy"]), c["vps"])
        base = I.Case("pencil", g, [I.Field(beam=I.beam_along_z(iso), spots=spots)], [I.Scenario()])
        per_spot = c["vps"]
    fields = []
    for f in base.fields:
        f = copy.copy(f)
        f.spots = s = f.spots.copy()
        n = len(s)
        s["x_mm"] += rng.normal(0.0, 0.2, n).astype(np.float32)
        s["y_mm"] += rng.normal(0.0, 0.2, n).astype(np.float32)
        s["weight"] = rng.uniform(0.5, 1.5, n).astype(np.float32)
        s["n_histories"] = (per_spot * rng.uniform(0.5, 1.5, n)).astype(np.uint32) if im else per_spot
        fields.append(f)
    return I.Case(base.name, base.geometry, fields, _scenarios(c["scenarios"], rng), seed=int(seed),
                  physics=c["physics"], n_batches=c.get("batches", 0))


def _steps_per_vp(c):
    """Condensed-history steps of a particle: the voxels of its range in the
    grid, about 15 steps of a quarter of the residual range at its end, and a
    few in the beam line."""
    if c["geom"] == "head":
        return 104.0 if c["target_cc"] == 8.0 else 94.0
    d = c["opening_mm"]
    through = (d / (d + 10.0)) ** 2 if d else 1.0   # share of the spots' particles in the opening
    e = c["energy"] if d == 0 else 147.0
    return through * (10.0 * 0.0022 * e ** 1.77 / c["mm"] + 18.0) + (10.0 if d else 0.0)


def _row_voxels(c):
    """Voxels that the particles of one influence-matrix row reach, about."""
    return 2200.0 * c["vps"] ** 0.36


# -------------------------------------------------- pencil-beam-like rows
def _row_problem(c, seed):
    """Rows (scenario, spot) on the GPU: each spot covers the voxels of a
    lateral square around its axis along +x down to its depth, values falling
    off laterally and rising towards the end; scenarios move the axes by up
    to a voxel.  Ascending voxels, some empty rows."""
    nx, ny, nz, n, S = c["nx"], c["ny"], c["nz"], c["spots"], c["scen"]
    # which voxels the rows reach is the grid's and the plan's; the seed gives the values
    rng = np.random.default_rng(nx * 1_000_003 + ny * 1009 + nz)
    jc, kc = rng.uniform(ny * 0.3, ny * 0.7, n), rng.uniform(nz * 0.3, nz * 0.7, n)
    hw = rng.integers(2, 6, n)
    depth = rng.integers(nx // 3, nx, n)
    depth[rng.choice(n, size=max(1, n // 50), replace=False)] = 0
    dj, dk = rng.uniform(-1.0, 1.0, (2, S))
    dj[0] = dk[0] = 0.0
    c0, c1 = (jc + dj[:, None]).ravel(), (kc + dk[:, None]).ravel()
    hwr, dr = np.tile(hw, S), np.tile(depth, S)
    j0, j1 = np.maximum(0, c0.astype(int) - hwr), np.minimum(ny, c0.astype(int) + hwr + 1)
    k0, k1 = np.maximum(0, c1.astype(int) - hwr), np.minimum(nz, c1.astype(int) + hwr + 1)
    lens = (j1 - j0) * (k1 - k0) * dr
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    rpd = t(rp)
    col = torch.empty(int(rp[-1]), dtype=torch.int32, device=dev)
    val = torch.empty(int(rp[-1]), dtype=torch.float32, device=dev)
    R = len(lens)
    for r0 in range(0, R, 2000):   # a slice of rows at a time: the temporaries stay small
        r1 = min(R, r0 + 2000)
        b, e = int(rp[r0]), int(rp[r1])
        if b == e:
            continue
        row = torch.repeat_interleave(torch.arange(r0, r1, device=dev), t(lens[r0:r1]))
        pos = torch.arange(b, e, device=dev) - rpd[row]
        d, wj = t(dr)[row], t(j1 - j0)[row]
        i, jj = pos % d, (pos // d)
        k, j = t(k0)[row] + jj // wj, t(j0)[row] + jj % wj
        col[b:e] = ((k * ny + j) * nx + i).to(torch.int32)
        w = 0.5 * t(hwr)[row].float()
        lat = torch.exp(-((j - t(c0)[row].float()) ** 2 + (k - t(c1)[row].float()) ** 2) / (2.0 * w * w))
        dep = 0.3 + 0.7 * (i.float() / torch.clamp(d - 1, min=1)) ** 4
        val[b:e] = 1e-3 * lat * dep * (0.9 + 0.2 * torch.rand(e - b, generator=g, device=dev))
    return rpd, col, val


@functools.lru_cache(maxsize=4)
def _structures(nx, ny, nz):
    """Target box in the middle, organ at risk a slab beside it; and the
    voxel -> cell map of dynamic spacing."""
    roi = np.zeros((nz, ny, nx), np.uint8)
    a, b, e = max(3, nz // 8), max(4, ny // 16), max(5, nx // 16)
    roi[nz // 2 - a: nz // 2 + a, ny // 2 - b: ny // 2 + b, nx // 2 - e: nx // 2 + e] |= 1
    roi[nz // 2 - a: nz // 2 + a, ny // 2 + b - 1: ny // 2 + 2 * b, nx // 3: nx] |= 2
    roi = roi.ravel()
    return (roi,) + I.dynamic_spacing_map((nx, ny, nz), roi)


OPT = dict(d_presc=2.0, w_target=1.0, d_max=0.8, w_oar=4.0)
CELL_K = 36   # fixed-point exponent of the merged energies


@functools.lru_cache(maxsize=2)
def _row_geometry(nx, ny, nz):
    """CT numbers of a grid of tissue with some bone and air."""
    h = np.random.default_rng(nx * 1_000_003 + ny * 1009 + nz).normal(30.0, 20.0, (nz, ny, nx))
    h[:, : ny // 10] = -1000.0
    h[:, ny // 10: ny // 8] = 1200.0
    return I.Geometry(I.GEOM_HU, (nx, ny, nz), HEAD_MM, (0.0, 0.0, 0.0), np.rint(h).astype(np.int16))


# --------------------------------------------------------------- surrogate
def _network_data(c, seed):
    """Entry states near an aperture's edge as the network sees them and
    outcomes of the kind brass gives: transmission falling with depth, loss,
    angle and offset around smooth functions of the state."""
    rng = np.random.default_rng(seed)
    m = c["n"] + c["held"]
    xy, ang, e = I.surrogate_training_entries(m, seed=seed)
    edge = np.abs(np.hypot(xy[:, 0], xy[:, 1]) - 10.0)
    x = np.column_stack([xy / 20.0, ang / 0.05, (e - 150.0) / 50.0, np.minimum(edge, 100.0) / 10.0, np.ones(m),
                         np.zeros(m)]).astype(np.float32)
    loss = np.clip(1.2 - (e - 70.0) / 160.0, 0.05, 1.0)
    y = np.column_stack([(loss + rng.normal(0, 0.05, m) - 0.5) / 0.25, np.abs(rng.normal(0.8, 0.3, m)),
                         np.abs(rng.normal(0.5, 0.25, m))]).astype(np.float32)
    t = (rng.uniform(size=m) < 1.0 / (1.0 + np.exp(6.0 * (loss - 0.6)))).astype(np.float32)
    y[t == 0] = 0.0
    return x, y, t


LR = 1e-3


# --------------------------------------------------------------- interface
def prepare(case, seed):
    c, kind = case, case["kind"]
    if kind in ("dose", "im"):
        plan = _case(c, seed)
        eng = V.Engine(0) if kind == "dose" else _engine_of(plan.geometry)
        eng.load_case(plan)
        s = {"case": c, "eng": eng, "plan": plan}
        if kind == "im":
            # the plan's matrix store, as large as its rows can need: every
            # pass leaves its entries in front and zeros behind them
            rows = len(plan.scenarios) * sum(len(f.spots) for f in plan.fields)
            n = int(rows * min(1.4 * _row_voxels(c), float(plan.geometry.nvox)))
            s["col"] = torch.zeros(n, dtype=torch.int32, device="cuda")
            s["val"] = torch.zeros(n, dtype=torch.float32, device="cuda")
        return s
    if kind == "surrogate":
        x, y, t = _network_data(c, seed)
        n = c["n"]
        return {"case": c, "eng": V.Engine(0), "x": x[:n], "y": y[:n], "t": t[:n], "held": x[n:],
                "w": V.surrogate_init(seed), "seed": int(seed)}
    rp, col, val = _row_problem(c, seed)
    roi, cmap, n_cells = _structures(c["nx"], c["ny"], c["nz"])
    dev = col.device
    s = {"case": c, "eng": V.Engine(0), "rp": rp, "col": col, "nvox": c["nx"] * c["ny"] * c["nz"]}
    if kind == "cells":
        V.vpmc_load_geometry(s["eng"].ctx, _row_geometry(c["nx"], c["ny"], c["nz"]))
        s["q"] = (val.double() * 2.0 ** CELL_K).to(torch.int64)
        s["map"], s["n_cells"] = torch.from_numpy(cmap).to(dev), n_cells
        return s
    s["val"], s["roi"] = val, torch.from_numpy(roi).to(dev)
    s["x0"] = torch.from_numpy(np.random.default_rng(seed + 1).uniform(40.0, 60.0, c["spots"])).to(dev)
    if c["reuse"]:   # re-planning: the index stands, the objective has changed
        s["eng"].optimize(rp, col, val, c["scen"], [c["spots"]], s["nvox"], s["roi"], iters=0, n_power=1, x0=s["x0"],
                          **OPT)
    return s


def run(s):
    c, eng = s["case"], s["eng"]
    if c["kind"] == "dose":
        sigma = c["batches"] >= 2
        dose, sig, led = eng.run_dose(s["plan"], 0, sigma=sigma, let=c["let"])
        if not c["let"]:
            return {"dose": dose, "sigma": sig, "ledger": led}
        let = [eng.last_let(i)[0] for i in range(c["scenarios"])]
        q = [eng.last_tally(i)[0] for i in range(c["scenarios"])]
        return {"dose": dose, "sigma": sig, "ledger": led, "let": let, "tally": q}
    if c["kind"] == "im":
        rp, col, val, _, k = eng.run_csr(s["plan"], device_out=True)
        s["col"][: len(col)].copy_(col)
        s["val"][: len(val)].copy_(val)
        return {"row_ptr": rp, "col": s["col"], "val": s["val"], "k": k, "ledger": eng.last_ledger}
    if c["kind"] == "optimize":
        x, L = eng.optimize(s["rp"], s["col"], s["val"], c["scen"], [c["spots"]], s["nvox"], s["roi"],
                            iters=c["iters"], x0=s["x0"], reuse=c["reuse"], **OPT)
        return {"x": x, "L": L[0]}
    if c["kind"] == "cells":
        rp, cell, q, val = V.vpmc_csr_cells(eng.ctx, s["rp"], s["col"], s["q"], CELL_K, s["map"], s["n_cells"],
                                            V.DEVICE_PTRS)
        return {"row_ptr": rp, "cell": cell, "q": q, "val": val}
    V.vpmc_surrogate_set_weights(eng.ctx, s["w"])
    loss = V.vpmc_surrogate_train(eng.ctx, s["x"], s["y"], s["t"], c["epochs"], c["batch"], LR, s["seed"])
    return {"loss": loss, "weights": V.vpmc_surrogate_get_weights(eng.ctx),
            "held": V.vpmc_surrogate_forward(eng.ctx, s["held"])}


def work(case):
    c, kind = case, case["kind"]
    if kind in ("dose", "im"):
        if c["geom"] == "head":
            nvox, ct = int(np.prod(HEAD)), 2
            spots = {0.4: 203, 8.0: 950}[c["target_cc"]] * c.get("fields", 1)
            vps = spots * c["vps"]
        else:
            nvox, ct = c["nx"] * c["ny"] * c["nz"], 0
            spots = {0: 1, 10: 49, 20: 113, 30: 197, 40: 317}[int(c["opening_mm"])]
            vps = c["vps"] * (spots if kind == "im" else 1)
        S = c["scenarios"]
        # about 300 arithmetic operations per condensed-history step (the method's own count)
        flops = 300.0 * _steps_per_vp(c) * vps * S
        if kind == "dose":
            per = 4 + (4 if c["batches"] >= 2 else 0) + (16 if c["let"] else 0)
            return {"bytes": float(nvox * (ct + per * S)), "flops": flops}
        return {"bytes": float(nvox * ct + 8.0 * min(_row_voxels(c), nvox) * spots * S), "flops": flops}
    if kind == "surrogate":
        p = 8 * 256 + 3 * 256 * 256 + 256 * 29
        n = c["n"] // c["batch"] * c["batch"] * c["epochs"]
        return {"bytes": 48.0 * c["n"] + 148.0 * c["held"] + 8.0 * p, "flops": 6.0 * p * n + 2.0 * p * c["held"]}
    # entries of the rows: mean (2 hw + 1)^2 of half widths 2..5, mean depth 2/3 nx
    entries = c["spots"] * c["scen"] * 69.0 * 0.667 * c["nx"]
    nvox = c["nx"] * c["ny"] * c["nz"]
    if kind == "cells":
        return {"bytes": entries * (12.0 + 16.0 * 0.3) + 4.0 * nvox, "flops": entries}
    used = 0.1 * entries   # in the structures' voxels
    sweeps = 2.0 * (c["iters"] + 20) + 1.0
    read = 0.0 if c["reuse"] else 8.0 * entries
    return {"bytes": read + 8.0 * used + nvox, "flops": 2.0 * used * sweeps}


# ------------------------------------------------------------ 64-bit values
def _exact_optimize(c, seed):
    rp, col, val = _row_problem(c, seed)
    roi = torch.from_numpy(_structures(c["nx"], c["ny"], c["nz"])[0]).to(col.device)
    n, S, dev = c["spots"], c["scen"], col.device
    inside = torch.nonzero(roi[col.long()]).ravel()
    row = torch.searchsorted(rp, inside, right=True) - 1
    vox = torch.nonzero(roi).ravel()
    index = torch.full((roi.numel(),), -1, dtype=torch.int64, device=dev)
    index[vox] = torch.arange(len(vox), device=dev)
    key = (row // n) * len(vox) + index[col[inside].long()]
    spot, a = row % n, val[inside].double()
    m = roi[vox].repeat(S)
    T, Or = (m & 1) > 0, (m & 2) > 0
    fwd = lambda w: torch.zeros(S * len(vox), dtype=torch.float64, device=dev).index_add_(0, key, a * w[spot])  # noqa: E731
    back = lambda r: torch.zeros(n, dtype=torch.float64, device=dev).index_add_(0, spot, a * r[key]) * (2.0 / S)  # noqa: E731
    z, lam = torch.ones(n, dtype=torch.float64, device=dev), 0.0
    M = OPT["w_target"] * T.double() + OPT["w_oar"] * Or.double()
    for _ in range(20):
        g = back(M * fwd(z))
        lam = float(g.norm() / z.norm())
        if float(g.norm()) > 0:
            z = g / g.norm()
    L = 1.05 * lam
    x = torch.from_numpy(np.random.default_rng(seed + 1).uniform(40.0, 60.0, n)).to(dev)
    y, t = x.clone(), 1.0
    for _ in range(c["iters"]):
        D = fwd(y)
        r = OPT["w_target"] * T * (D - OPT["d_presc"]) + OPT["w_oar"] * Or * torch.clamp(D - OPT["d_max"], min=0.0)
        xn = torch.clamp(y - back(r) / L if L > 0 else y, min=0.0)
        tn = 0.5 * (1.0 + math.sqrt(1.0 + 4.0 * t * t))
        y, x, t = xn + (t - 1.0) / tn * (xn - x), xn, tn
    return {"x": x, "L": L}


def _exact_cells(c, seed):
    rp, col, val = _row_problem(c, seed)
    _, cmap, n_cells = _structures(c["nx"], c["ny"], c["nz"])
    g = _row_geometry(c["nx"], c["ny"], c["nz"])
    dev = col.device
    cm = torch.from_numpy(cmap).to(dev)
    rho = np.interp(np.clip(g.hu, -1000, 3071).ravel(), [-1000.0, 0.0, 1000.0, 1500.0, 3071.0],
                    [0.00121, 1.0, 1.6, 1.85, 2.8])
    mass = torch.zeros(n_cells, dtype=torch.float64, device=dev).index_add_(0, cm.long(), torch.from_numpy(rho).to(dev))
    mass *= float(np.prod(np.asarray(g.spacing, np.float64))) * 1e-6
    q = (val.double() * 2.0 ** CELL_K).to(torch.int64)
    cell = cm[col.long()]
    start = torch.ones(len(col), dtype=torch.bool, device=dev)
    start[1:] = cell[1:] != cell[:-1]
    start[rp[:-1][rp[:-1] < len(col)]] = True
    at = torch.cumsum(start, 0) - 1
    sums = torch.zeros(int(at[-1]) + 1, dtype=torch.int64, device=dev).index_add_(0, at, q)
    cells = cell[start]
    before = torch.zeros(len(col) + 1, dtype=torch.int64, device=dev)
    before[1:] = torch.cumsum(start, 0)
    v = sums.double() * (1.602176634e-13 * 2.0 ** -CELL_K) / mass[cells.long()]
    return {"row_ptr": before[rp], "cell": cells, "q": sums, "val": v}


def _exact_surrogate(c, seed):
    dims, n, B = V.SURROGATE_DIMS, c["n"], c["batch"]
    xs, ys, ts = _network_data(c, seed)
    dev = torch.device("cuda")
    X, Y, T = (torch.from_numpy(a).to(dev).double() for a in (xs, ys, ts))
    flat = torch.from_numpy(V.surrogate_init(seed)).to(dev).double()
    ps, o = [], 0
    for ni, no in zip(dims[:-1], dims[1:]):
        ps += [flat[o:o + ni * no].reshape(no, ni).clone(), flat[o + ni * no:o + ni * no + no].clone()]
        o += ni * no + no
    for p in ps:
        p.requires_grad_(True)

    def net(h):
        for l in range(len(dims) - 1):
            h = h @ ps[2 * l].t() + ps[2 * l + 1]
            h = torch.nn.functional.silu(h) if l < len(dims) - 2 else h
        return h

    opt = torch.optim.Adam(ps, lr=float(np.float32(LR)), betas=(0.9, 0.999), eps=1e-8)
    st, mask, losses = int(seed) ^ 0x9E3779B97F4A7C15, (1 << 64) - 1, []
    for _ in range(c["epochs"]):
        perm = list(range(n))   # the shuffle of the training call
        for i in range(n - 1, 0, -1):
            st ^= st >> 12
            st ^= (st << 25) & mask
            st ^= st >> 27
            j = (((st * 0x2545F4914F6CDD1D) & mask) >> 11) % (i + 1)
            perm[i], perm[j] = perm[j], perm[i]
        p = torch.tensor(perm, device=dev)
        tot, nb = 0.0, 0
        for s0 in range(0, n - B + 1, B):
            b = p[s0:s0 + B]
            out, y, t = net(X[b]), Y[b], T[b]
            bce = torch.nn.functional.binary_cross_entropy_with_logits(out[:, 0], t, reduction="none")
            mu, ls = out[:, 5:17].reshape(-1, 4, 3), out[:, 17:29].reshape(-1, 4, 3)
            lp = (-0.5 * ((y[:, None] - mu) * torch.exp(-ls)) ** 2 - ls - 0.5 * math.log(2.0 * math.pi)).sum(2)
            nll = -torch.logsumexp(torch.log_softmax(out[:, 1:5], 1) + lp, 1)
            loss = (bce + torch.where(t > 0.5, nll, torch.zeros_like(nll))).mean()
            opt.zero_grad()
            loss.backward()
            opt.step()
            tot, nb = tot + float(loss.detach()), nb + 1
        losses.append(tot / nb if nb else 0.0)
    with torch.no_grad():
        held = net(X[n:])
    return {"loss": np.array(losses), "weights": torch.cat([p.detach().ravel() for p in ps]), "held": held}


def exact(case, seed):
    return {"optimize": _exact_optimize, "cells": _exact_cells, "surrogate": _exact_surrogate}.get(
        case["kind"], lambda c, s: None)(case, seed)
