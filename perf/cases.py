"""Timed cases of the library: what a control plane built on it calls, over the sizes it calls with.

Every case goes through the binding's Device* objects, which a program builds once per set of
inputs (tables, fleet state and requests copied to the GPU, outputs and workspace allocated)
and then calls.  Inputs are drawn by paper_2606_30391_amd.workloads from the given seed.
``exact`` evaluates the same definitions (include/festina.h) in float64 with plain torch.

Case fields: "path" names the call; the sizes are the workload's.
"""
import math

import numpy as np
import torch

from paper_2606_30391_amd import festina, workloads

N_ROWS = 32
# GPUs hosting one model, as a share of the fleet, per placement law (config): all models on
# every GPU; 2 of 8; 1-4 of 32; 1-4 of 32
HOST_SHARE = {1: 1.0, 2: 0.25, 3: 2.5 / 32, 4: 2.5 / 32}
MODELS = {1: 2, 2: 8, 3: 32, 4: 32}
CELLS = {1: 32, 2: 128, 3: 128, 4: 128}
# configuration 4 caps prefill and decode at 2, 4 or 6 of 8 SM levels: a GPU's distinct cells
CAPPED_SHARE = 44.0 / 72.0


def listed():
    return [
        # --- the batched placement search (the framework's main path)
        # the smallest call: a handful of pending requests on one 8-GPU node, 4 x 8 levels,
        # through the allocation-free entry point a serving loop uses
        {"name": "place-node", "path": "place", "config": 1, "requests": 64, "gpus": 8, "noalloc": True},
        # a rack: 4,096 requests on 64 GPUs with two models each
        {"name": "place-rack", "path": "place", "config": 2, "requests": 4096, "gpus": 64, "noalloc": False},
        # odd sizes of the capped, bursty law (several arrival waves, partly filled tiles)
        {"name": "place-odd", "path": "place", "config": 4, "requests": 20011, "gpus": 333, "noalloc": True},
        # a large fleet in one arrival wave, no SM caps, a tenth of the requests infeasible
        {"name": "place-fleet", "path": "place", "config": 3, "requests": 65536, "gpus": 512, "noalloc": False},
        # the benchmark's placement: 64 arrival waves of 4,096 requests, phase-aware SM caps
        {"name": "place-bursts", "path": "place", "config": 4, "requests": 262144, "gpus": 1024, "noalloc": False},
        # --- consolidation and the schedulers around the search
        # every ordered pair of a 2,048-GPU fleet (the benchmark's consolidation)
        {"name": "migrate", "path": "migrate", "gpus": 2048},
        # the local schedulers' joint SM/frequency sweep: 1,024 GPUs x 64 epochs of batches
        {"name": "sweep", "path": "sweep", "gpus": 1024, "epochs": 64, "tasks": 8, "per_batch": False},
        # preferred configuration of every instance, then the fleet's energy waste ratio
        {"name": "preferred", "path": "preferred", "gpus": 2048},
        # the paper's dispatcher: one request against 10,000 GPUs (its scheduler-latency table)
        {"name": "dispatch-one", "path": "dispatch", "requests": 1, "gpus": 10000},
        # the dispatcher on a burst against one snapshot
        {"name": "dispatch-burst", "path": "dispatch", "requests": 65536, "gpus": 512},
        # the dispatcher over 64 arrival waves, each committed before the next
        {"name": "dispatch-waves", "path": "waves", "requests": 262144, "gpus": 1024, "waves": 64},
        # the transfer plan of a reconfiguration: cost matrix and per-request moves
        {"name": "transfer", "path": "transfer", "gpus": 2048, "per_gpu": 8},
    ]


def _log_int(rng, lo, hi):
    """Whole number, log-uniform over [lo, hi], odd ones as likely as even ones."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges; the main path twice as often as each other one."""
    path = rng.choice(["place", "place", "place", "place", "migrate", "sweep", "preferred", "dispatch", "waves",
                       "transfer"])
    if path == "place":
        config = rng.choice([1, 2, 3, 4])
        lo, hi = {1: (8, 1024), 2: (256, 16384), 3: (4096, 65536), 4: (8192, 262144)}[config]
        glo, ghi = {1: (2, 32), 2: (16, 256), 3: (64, 512), 4: (128, 1024)}[config]
        return {"path": path, "config": config, "requests": _log_int(rng, lo, hi), "gpus": _log_int(rng, glo, ghi),
                "noalloc": rng.random() < 0.5}
    if path == "migrate":
        return {"path": path, "gpus": _log_int(rng, 64, 2048)}
    if path == "sweep":
        return {"path": path, "gpus": _log_int(rng, 16, 1024), "epochs": _log_int(rng, 2, 64),
                "tasks": rng.choice([4, 8, 12, 16]), "per_batch": rng.random() < 0.5}
    if path == "preferred":
        return {"path": path, "gpus": _log_int(rng, 32, 2048)}
    if path == "dispatch":
        gpus = _log_int(rng, 64, 10000)
        return {"path": path, "requests": _log_int(rng, 1, min(65536, 65536 * 512 // gpus)), "gpus": gpus}
    if path == "waves":
        waves = _log_int(rng, 4, 64)
        return {"path": path, "requests": waves * _log_int(rng, 64, 4096) + rng.randrange(waves),
                "gpus": _log_int(rng, 128, 1024), "waves": waves}
    return {"path": path, "gpus": _log_int(rng, 64, 2048), "per_gpu": rng.choice([2, 5, 8])}


# ------------------------------------------------------------------ inputs, call, work
def _inputs(case, seed):
    path, seed = case["path"], int(seed)
    if path == "place":
        return workloads.make_placement(case["config"], seed=seed, n_requests=case["requests"], n_gpus=case["gpus"])
    if path == "migrate":
        return workloads.make_fleet(seed=seed, n_gpus=case["gpus"])
    if path == "sweep":
        inp = workloads.make_sweep(seed=seed, n_gpus=case["gpus"], n_epochs=case["epochs"], max_tasks=case["tasks"])
        inp["batches"]["static_power"] = 1 if case["per_batch"] else 0
        return inp
    if path == "preferred":
        return workloads.make_llms(seed=seed, n_gpus=case["gpus"])
    if path == "dispatch":
        return workloads.make_dispatch(seed=seed, n_requests=case["requests"], n_gpus=case["gpus"])
    if path == "waves":
        return workloads.make_dispatch_waves(seed=seed, n_requests=case["requests"], n_gpus=case["gpus"],
                                             n_waves=case["waves"])
    return workloads.make_transfer(seed=seed, n_gpus=case["gpus"], requests_per_gpu=case["per_gpu"])


def prepare(case, seed):
    """The device object a program holds before the call."""
    inp = _inputs(case, seed)
    path = case["path"]
    cls = {"place": festina.DevicePlacement, "migrate": festina.DeviceMigration, "sweep": festina.DeviceSweep,
           "preferred": festina.DevicePreferred, "dispatch": festina.DeviceDispatch, "waves": festina.DeviceDispatch,
           "transfer": festina.DeviceTransfer}[path]
    return {"path": path, "dev": cls(inp, "cuda"), "noalloc": case.get("noalloc", False),
            "wave_start": inp.get("wave_start")}


def run(state):
    """One pass; the outputs are the object's own buffers."""
    d, path = state["dev"], state["path"]
    if path == "place":
        if state["noalloc"]:
            d.run_noalloc()
        else:
            d.run()
        return {"choice": d.choice, "feasible": d.feasible, "energy": d.energy}
    if path == "migrate":
        d.run()
        return {"best_dst": d.best_dst, "saving": d.saving, "level": d.level}
    if path == "sweep":
        d.run()
        return {"level": d.level, "feasible": d.feasible, "energy": d.energy, "task_sm": d.task_sm}
    if path == "preferred":
        d.run()
        out = dict(d.o)
        out.update(f_gpu=d.f_gpu, waste_gpu=d.waste_gpu, totals=d.totals)
        return out
    if path == "dispatch":
        d.run()
        return dict(d.o)
    if path == "waves":
        d.run_waves(state["wave_start"])
        out = dict(d.o)
        out.update(("state_" + k, v) for k, v in d.state_t.items())
        return out
    d.run_costs()
    d.run_moves()
    return {"cost": d.cost, "decision": d.decision, "remaining": d.remaining, "migrate": d.migrate}


def work(case):
    """Inputs read once and outputs written once; the operations on the candidates (a multiply,
    an add and a comparison per placement candidate, and so on for the others)."""
    path, g = case["path"], case["gpus"]
    tables = 2 * 32 * N_ROWS * 128 * 4
    if path == "place":
        c, r = case["config"], case["requests"]
        waves = 64 if c == 4 else 1
        cand = r * HOST_SHARE[c] * g * CELLS[c] * (CAPPED_SHARE if c == 4 else 1.0)
        data = r * (24 + 9) + waves * g * 4 + g * 10 + 2 * MODELS[c] * N_ROWS * CELLS[c] * 4
        return {"bytes": float(data), "flops": 3.0 * cand}
    if path == "migrate":
        return {"bytes": float(g * (4 * 6 * 4 + 20 + 12) + tables), "flops": 8.0 * g * (g - 1)}
    if path == "sweep":
        b = g * case["epochs"]
        tasks = 2.45 * b
        return {"bytes": float(b * (12 + 9 + 4 * case["tasks"]) + tasks * 16 + tables), "flops": tasks * 128 + tasks * 16 * 5}
    if path == "preferred":
        return {"bytes": float(4 * g * (6 * 4 + 11 * 4 + 1) + g * 20 + tables), "flops": 2.5 * g * 256 * 5}
    if path in ("dispatch", "waves"):
        r, w = case["requests"], case.get("waves", 1)
        pts = r * HOST_SHARE[4] * g
        return {"bytes": float(r * (20 + 17) + w * g * (16 + 4 * 12) + tables), "flops": pts * 20}
    q = g * case["per_gpu"]
    return {"bytes": float(4 * g * g + g * 28 + q * 36 + tables), "flops": 3.0 * g * g}


def tolerance(case):
    """Four times the distance from float64 measured over these ranges: energies and savings are
    float32 sums of a few terms (a GPU's energy waste is a difference of near values), levels,
    choices and destinations may differ where two candidates lie within rounding."""
    path = case["path"]
    if path in ("dispatch", "waves", "transfer"):
        return "exact"               # evaluated in float64 in a stated order, rounded once
    if path == "preferred":
        return {"rel": 2e-6, "max": 1.5e-5, "differ": 1e-4}
    if path == "migrate":
        return {"rel": 4e-7, "max": 1.2e-6, "differ": 4e-3}
    return {"rel": 2e-7, "max": 8e-7, "differ": 1e-4}


# ------------------------------------------------------------------ float64 evaluation
def _t(a, dtype):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda" if torch.cuda.is_available() else "cpu").to(dtype)


F32, F64, I64 = torch.float32, torch.float64, torch.int64


def _prompt_row(tokens):
    return torch.clamp((tokens + 255) // 256, max=N_ROWS) - 1


def _resident(bits, m):
    b = _t(np.asarray(bits, np.uint32).astype(np.int64), I64)
    ids = torch.arange(m, device=b.device)
    return ((b[:, ids // 32] >> (ids % 32)) & 1).bool()              # [G][M]


def _first_min(e, index, none):
    """Least value along the last axis and the least index among its ties; `none` where all inf."""
    v = e.min(dim=-1).values
    i = torch.where((e == v[..., None]) & torch.isfinite(e), index, torch.iinfo(I64).max).min(dim=-1).values
    found = torch.isfinite(v)
    return v, torch.where(found, i, torch.full_like(i, none)), found


def _exact_place(inp):
    lut, gp, rq = inp["lut"], inp["gpus"], inp["requests"]
    M, NS, NF, G, W, R = (lut["n_models"], lut["n_sm"], lut["n_freq"], gp["n_gpus"], gp["n_waves"], rq["n_requests"])
    pf, dc = _t(lut["pf"], F32), _t(lut["dc"], F32)
    dev = pf.device
    s, f = _t(lut["sm_level"], F64), _t(lut["freq_level"], F64)
    batch, kd, res = _t(gp["batch"], I64).reshape(W, G), _t(gp["k_dyn_w"], F64), _resident(gp["resident"], M)
    top = torch.full((G,), NS - 1, dtype=I64, device=dev)
    cp = top if gp["cap_pf"] is None else _t(gp["cap_pf"], I64)
    cd = top if gp["cap_dc"] is None else _t(gp["cap_dc"], I64)
    model, wave = rq["model"], rq["wave"] if rq["wave"] is not None else np.zeros(R, np.int32)
    prompt, pred = _t(rq["prompt_tokens"], I64), _t(rq["pred_out_tokens"], I64)
    lout = ((pred * 105 + 99) // 100).to(F64)
    st, sb = _t(rq["slo_ttft_ms"], F32), _t(rq["slo_tbt_ms"], F32)
    choice = torch.full((R,), -1, dtype=I64, device=dev)
    energy = torch.full((R,), math.inf, dtype=F64, device=dev)
    js, fk = torch.arange(NS, device=dev), f * f * f
    order = np.lexsort((model, wave))
    key = wave[order].astype(np.int64) * M + model[order]
    cut = np.flatnonzero(np.diff(key)) + 1
    for part in np.split(order, cut):
        if not len(part):
            continue
        m, w = int(model[part[0]]), int(wave[part[0]])
        hosts = torch.nonzero(res[:, m]).reshape(-1)
        if not len(hosts):
            continue
        b = torch.clamp(batch[w, hosts] + 1, max=N_ROWS)
        kap = kd[hosts] * b.to(F64) / 32.0
        jp, jd = torch.minimum(js[None], cp[hosts, None]), torch.minimum(js[None], cd[hosts, None])   # [H][NS]
        pp = lut["p0_w"] + kap[:, None, None] * s[jp][:, :, None] * fk
        pd = lut["p0_w"] + kap[:, None, None] * s[jd][:, :, None] * fk
        tbt = dc[m][b - 1].gather(1, jd[:, :, None].expand(-1, -1, NF))                               # [H][NS][NF]
        y = pd * tbt.to(F64)
        idx = ((hosts[:, None, None] * NS + js[None, :, None]) * NF + torch.arange(NF, device=dev)).reshape(-1)
        step = max(1, 60_000_000 // idx.numel())
        for r in torch.from_numpy(part).to(dev).split(step):
            row = torch.where(prompt[r][:, None] > 0, _prompt_row(prompt[r])[:, None], b[None] - 1)    # [n][H]
            if bool((prompt[r] > 0).all()):
                t = pf[m][_prompt_row(prompt[r])][:, jp]                                               # [n][H][NS][NF]
            else:
                t = pf[m][row].gather(2, jp[None, :, :, None].expand(len(r), -1, -1, NF))
            e = pp * t.to(F64) + lout[r][:, None, None, None] * y
            ok = (t < st[r][:, None, None, None]) & (tbt < sb[r][:, None, None, None])
            e = torch.where(ok, e, math.inf).reshape(len(r), -1)
            energy[r], choice[r], _ = _first_min(e, idx, -1)
    return {"choice": choice, "feasible": torch.isfinite(energy).to(torch.uint8), "energy": energy}


def _exact_migrate(inp):
    lut, fl = inp["lut"], inp["fleet"]
    M, NS, NF, G, K = lut["n_models"], lut["n_sm"], lut["n_freq"], fl["n_gpus"], fl["max_inst"]
    pf, dc, f = _t(lut["pf"], F32), _t(lut["dc"], F32), _t(lut["freq_level"], F64)
    n, m, b, j = (_t(fl[k], I64) for k in ("n_inst", "inst_model", "inst_batch", "inst_sm"))
    brow = torch.clamp(b + 1, max=N_ROWS) - 1
    pt = _t(fl["inst_prompt_tokens"], I64)
    row = torch.where(pt > 0, _prompt_row(pt), brow)
    ok = (pf[m, row, j] < _t(fl["inst_slo_ttft_ms"], F32)[..., None]) & \
         (dc[m, brow, j] < _t(fl["inst_slo_tbt_ms"], F32)[..., None])                                  # [G][K][NF]
    ok |= (torch.arange(K, device=n.device)[None] >= n[:, None])[..., None]
    lev = ok.all(dim=1)                                                                                # [G][NF]
    hbm, sm = _t(fl["hbm_mib"], I64), _t(fl["sm_permille"], I64)
    u, kd = _t(fl["util"], F64), _t(fl["k_dyn_w"], F64)
    f3 = f * f * f
    both = lev[:, None] & lev[None]
    k = torch.argmax(both.to(torch.int32), dim=-1)                                                     # lowest common
    k0 = torch.argmax(lev.to(torch.int32), dim=-1)
    pair = both.any(dim=-1) & (hbm[:, None] + hbm[None] <= fl["hbm_cap_mib"]) & \
        (sm[:, None] + sm[None] <= fl["sm_cap_permille"]) & ~torch.eye(G, dtype=torch.bool, device=n.device)
    save = lut["p0_w"] - kd[None] * (f3[k] * (u[:, None] + u[None]) - f3[k0][None] * u[None])
    v, d, found = _first_min(torch.where(pair, -save, math.inf), torch.arange(G, device=n.device), -1)
    level = torch.where(found, k.gather(1, d.clamp(min=0)[:, None])[:, 0], -1)
    return {"best_dst": d, "saving": -v, "level": level}


def _exact_sweep(inp):
    lut, bt = inp["lut"], inp["batches"]
    NS, NF, B, T = lut["n_sm"], lut["n_freq"], bt["n_batches"], bt["max_tasks"]
    tab = torch.stack([_t(lut["pf"], F32), _t(lut["dc"], F32)])
    dev = tab.device
    s, f = _t(lut["sm_level"], F64), _t(lut["freq_level"], F64)
    units, ks = _t(bt["sm_units"], I64), torch.arange(NF, device=dev)
    out = [[], [], [], []]
    for b in torch.arange(B).split(4096):
        b = b.numpy()
        n, m, ph, tok = (_t(bt[k][b], I64) for k in ("n_tasks", "task_model", "task_phase", "task_tokens"))
        row = torch.where(ph == 0, _prompt_row(tok.clamp(min=1)), torch.clamp(tok, 1, N_ROWS) - 1)
        lat = tab[ph, m, row]                                                                          # [b][T][NS][NF]
        below = lat < _t(bt["task_slack_ms"][b], F32)[:, :, None, None]
        used = (torch.arange(T, device=dev)[None] < n[:, None])[..., None]
        has, j = below.any(dim=2), torch.argmax(below.to(torch.int32), dim=2)                          # [b][T][NF]
        t = torch.where(used & has, lat.gather(2, j[:, :, None])[:, :, 0].to(F64), 0.0)
        ku = (_t(bt["k_dyn_w"][b], F64) * _t(bt["util"][b], F64))[:, None] * (f * f * f)               # [b][NF]
        per_batch = bt["static_power"] == 1
        e = (((0.0 if per_batch else lut["p0_w"]) + ku[:, None] * s[j]) * t).sum(dim=1)
        if per_batch:
            e = e + lut["p0_w"] * t.max(dim=1).values
        share = torch.where(used, units[j], 0).sum(dim=1)
        ok = (has | ~used).all(dim=1) & (share < bt["sm_budget"])
        v, k, found = _first_min(torch.where(ok, e, math.inf), ks, -1)
        js = j.gather(2, k.clamp(min=0)[:, None, None].expand(-1, T, 1))[:, :, 0]
        for o, x in zip(out, (k, found.to(torch.uint8), v, torch.where(used[..., 0] & found[:, None], js, -1))):
            o.append(x)
    return dict(zip(("level", "feasible", "energy", "task_sm"), (torch.cat(o) for o in out)))


def _exact_preferred(inp):
    lut, q = inp["lut"], inp["llms"]
    NS, NF, G, K = lut["n_sm"], lut["n_freq"], q["n_gpus"], q["max_inst"]
    s, f = _t(lut["sm_level"], F64), _t(lut["freq_level"], F64)
    n, m, tin, tout, b = (_t(q[k], I64) for k in ("n_inst", "model", "avg_in_tokens", "avg_out_tokens", "batch"))
    used = (torch.arange(K, device=n.device)[None] < n[:, None]) & (tin >= 1)
    brow = torch.clamp(b + 1, max=N_ROWS) - 1
    ku = _t(q["k_dyn_w"], F64)[:, None] * (brow + 1).to(F64) / 32.0
    p = lut["p0_w"] + ku[..., None, None] * s[:, None] * (f * f * f)                                   # [G][K][NS][NF]
    cells = torch.arange(NS * NF, device=n.device)
    o = {}
    for x, tab, row, slo, scale in (("p", "pf", _prompt_row(tin.clamp(min=1)), "slo_ttft_ms", None),
                                    ("d", "dc", brow, "slo_tbt_ms", tout)):
        lat = _t(lut[tab], F32)[m, row]
        dur = lat.to(F64) if scale is None else lat.to(F64) * scale[..., None, None]
        ok = (lat < _t(q[slo], F32)[..., None, None]) & used[..., None, None]
        _, c, found = _first_min(torch.where(ok, p * dur, math.inf).reshape(G, K, -1), cells, -1)
        at = c.clamp(min=0)[..., None]
        o["sm_" + x] = torch.where(found, c // NF, -1)
        o["f_" + x] = torch.where(found, c % NF, -1)
        o["t_%s_ms" % x] = torch.where(found, dur.reshape(G, K, -1).gather(2, at)[..., 0], 0.0)
        o["p_%s_w" % x] = torch.where(found, p.reshape(G, K, -1).gather(2, at)[..., 0], 0.0)
    o["t_ms"] = o["t_p_ms"] + o["t_d_ms"]
    both = (o["sm_p"] >= 0) & (o["sm_d"] >= 0)
    tp, td = o["t_p_ms"], o["t_d_ms"]
    ep, ed = o["p_p_w"] * tp, o["p_d_w"] * td
    nan = torch.full_like(tp, math.nan)
    o["sm_pref"] = torch.where(both, (s[o["sm_p"].clamp(min=0)] * tp + s[o["sm_d"].clamp(min=0)] * td) / (tp + td), nan)
    o["f_pref"] = torch.where(both, (ep * f[o["f_p"].clamp(min=0)] + ed * f[o["f_d"].clamp(min=0)]) / (ep + ed), nan)
    o["feasible"] = both.to(torch.uint8)
    fp = torch.where(both, o["f_pref"], 0.0)
    fg = fp.max(dim=1).values
    t = torch.where(both, o["t_ms"], 0.0)
    waste = (t * (fg[:, None] ** 3 - fp ** 3)).sum(dim=1)
    best = (t * fp ** 3).sum()
    o = {k: v.reshape(-1) for k, v in o.items()}
    o.update(f_gpu=fg, waste_gpu=waste, totals=torch.stack([waste.sum(), best, waste.sum() / best]))
    return o


class _Dispatcher:
    """The current-frequency dispatcher on a state of the GPUs, dense over (request, GPU)."""

    def __init__(self, inp):
        lut, av, rq = inp["lut"], inp["avail"], inp["requests"]
        self.NS, self.NF, self.p0, self.k_new = lut["n_sm"], lut["n_freq"], float(np.float32(lut["p0_w"])), av["k_new_w"]
        self.pf, self.dc = _t(lut["pf"], F32), _t(lut["dc"], F32)
        self.s, self.f = _t(lut["sm_level"], F64), _t(lut["freq_level"], F64)
        self.freq, self.batch, self.mem, self.sm = (_t(av[k], I64) for k in ("freq_cur", "batch", "mem_free_mib",
                                                                             "sm_free"))
        self.kd, self.ta, self.kv = _t(av["k_dyn_w"], F64), _t(av["t_avail_ms"], F64), _t(av["kv_kib_per_token"], I64)
        self.res = _resident(av["resident"], lut["n_models"])
        self.m, self.prompt = _t(rq["model"], I64), _t(rq["prompt_tokens"], I64)
        self.lout = (_t(rq["pred_out_tokens"], I64) * 105 + 99) // 100
        self.st, self.sb = _t(rq["slo_ttft_ms"], F32), _t(rq["slo_tbt_ms"], F32)

    def _point(self, r, b, j, k, ta, kd):
        """Energy of each operating point, inf where it misses an SLO or has no SM level."""
        m = self.m[r][:, None]
        row = torch.where(self.prompt[r] > 0, _prompt_row(self.prompt[r]), -1)[:, None]
        row = torch.where(row >= 0, row, b - 1)
        jc = j.clamp(min=0)
        ttft, tbt = self.pf[m, row, jc, k], self.dc[m, b - 1, jc, k]
        power = self.p0 + kd * self.s[jc] * (self.f[k] * self.f[k] * self.f[k]) * (b.to(F64) / 32.0)
        e = power * (ttft.to(F64) + self.lout[r][:, None].to(F64) * tbt.to(F64))
        ok = (j >= 0) & (ta + ttft.to(F64) < self.st[r][:, None].to(F64)) & (tbt < self.sb[r][:, None])
        return torch.where(ok, e, math.inf)

    def run(self, r):
        """Results of requests r against the current state: gpu, freq, sm, phase, energy, step, need."""
        dev, G = self.m.device, len(self.batch)
        ids = torch.arange(G, device=dev)
        need = self.kv[self.m[r]] * (self.prompt[r] + self.lout[r])
        holds = self.mem[None] * 1024 >= need[:, None, None]                                           # [n][G][S]
        step = torch.argmax(holds.to(torch.int32), dim=2)
        cand = holds.any(dim=2) & self.res[:, self.m[r]].T
        ta, sm, mem = (x[ids[None], step] for x in (self.ta, self.sm, self.mem))
        b = torch.clamp(self.batch + 1, max=N_ROWS)[None].expand(len(r), -1)
        kd, kcur = self.kd[None], self.freq[None].expand(len(r), -1)
        e = torch.where(cand, self._point(r, b, sm, kcur, ta, kd), math.inf)
        emin = e.min(dim=1).values
        key = (mem << 32) | ((sm & 0xff) << 24) | (0xffffff - ids[None])
        key = torch.where(torch.isfinite(e) & (e <= (emin + 0.02 * emin.abs())[:, None]), key, torch.iinfo(I64).min)
        g1 = key.argmax(dim=1)
        p1 = torch.isfinite(emin)
        top = torch.full_like(kcur, self.NF - 1)
        e2 = torch.where(cand, self._point(r, b, sm, top, ta, kd), math.inf)
        _, g2, p2 = _first_min(torch.where(torch.isfinite(e2), ta, math.inf), ids, -1)
        ks = torch.arange(self.NF, device=dev)[None].expand(len(r), -1)
        e3, k3, p3 = _first_min(self._point(r, torch.ones_like(ks), torch.full_like(ks, self.NS - 1), ks,
                                            torch.zeros_like(ks).to(F64), self.k_new), ks[0], -1)
        g = torch.where(p1, g1, g2)
        gc, n = g.clamp(min=0), torch.arange(len(r), device=dev)
        on = p1 | p2
        phase = torch.where(p1, 1, torch.where(p2, 2, torch.where(p3, 3, 0)))
        freq = torch.where(p1, kcur[n, gc], torch.where(p2, self.NF - 1, k3))
        lev = torch.where(on, sm[n, gc], torch.where(p3, self.NS - 1, -1))
        en = torch.where(p1, e[n, gc], torch.where(p2, e2[n, gc], e3))
        return torch.where(on, g, -1), freq, lev, phase.to(torch.uint8), en, step[n, gc], need

    def commit(self, g, phase, step, need):
        on = g >= 0
        g, step, mib = g[on], step[on], (need[on] + 1023) // 1024
        self.batch.index_add_(0, g, torch.ones_like(g))
        self.freq[g[phase[on] == 2]] = self.NF - 1
        S = self.mem.shape[1]
        taken = torch.zeros_like(self.mem)
        for k in range(S):
            taken[:, k].index_add_(0, g, torch.where(step <= k, mib, 0))
        self.mem = torch.clamp(self.mem - taken, min=-1)


DISPATCH_OUT = ("gpu", "freq_level", "sm_level", "phase", "energy_mj")


def _exact_dispatch(inp):
    d = _Dispatcher(inp)
    R = inp["requests"]["n_requests"]
    parts = [d.run(r)[:5] for r in torch.arange(R, device=d.m.device).split(max(1, 8_000_000 // len(d.batch)))]
    return dict(zip(DISPATCH_OUT, (torch.cat(x) for x in zip(*parts))))


def _exact_waves(inp):
    d = _Dispatcher(inp)
    parts = []
    for lo, hi in zip(inp["wave_start"][:-1], inp["wave_start"][1:]):
        if hi > lo:
            o = d.run(torch.arange(int(lo), int(hi), device=d.m.device))
            d.commit(o[0], o[3], o[5], o[6])
            parts.append(o[:5])
    out = dict(zip(DISPATCH_OUT, (torch.cat(x) for x in zip(*parts))))
    out.update(state_freq_cur=d.freq, state_batch=d.batch, state_mem_free_mib=d.mem.reshape(-1))
    return out


def _exact_transfer(inp):
    lut, tr, pl, mv = inp["lut"], inp["transfer"], inp["plan"], inp["moves"]
    res = _resident(tr["resident"], inp["n_models"]).to(F64)
    mib = _t(tr["state_mib"], F64)[:, None] + (res * _t(tr["weights_mib"], F64)) @ (1.0 - res).T.contiguous()
    node = _t(tr["node"], I64)
    per = lambda same: torch.where(same, 1e3 / (float(np.float32(tr["bw_intra_gbs"])) * 1e9),
                                   1e3 / (float(np.float32(tr["bw_inter_gbs"])) * 1e9)).to(F64)
    cost = mib * 1048576.0 * per(node[:, None] == node[None])
    cost.fill_diagonal_(0.0)
    src, m, ctx, rem, kv, tok = (_t(mv[k], I64) for k in ("src", "model", "context_tokens", "remaining_tokens",
                                                          "kv_kib", "token_kib"))
    dest, freq, sm, batch = (_t(pl[k], I64) for k in ("dest", "freq_cur", "sm_cur", "batch"))
    v = dest[src]
    left = rem.to(F64) * _t(lut["dc"], F64)[m, torch.clamp(batch[src] + 1, max=N_ROWS) - 1, sm[src], freq[src]]
    link = per(node[src] == node[v])
    t_kv, t_tok = kv.to(F64) * 1024.0 * link, tok.to(F64) * 1024.0 * link
    t_rec = _t(lut["pf"], F64)[m, _prompt_row(ctx), sm[v], freq[v]]
    move = torch.where(v != src, t_tok + torch.minimum(t_kv, t_rec), 0.0)
    dec = torch.where((v != src) & (left > move), torch.where(t_kv < t_rec, 1, 2), 0)
    return {"cost": cost, "decision": dec, "remaining": left, "migrate": move}


def exact(case, seed):
    """run()'s outputs in float64, laid out the same."""
    return {"place": _exact_place, "migrate": _exact_migrate, "sweep": _exact_sweep, "preferred": _exact_preferred,
            "dispatch": _exact_dispatch, "waves": _exact_waves, "transfer": _exact_transfer}[case["path"]](
                _inputs(case, seed))
