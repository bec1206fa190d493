"""The work a user has the library do, as cases that can be timed and compared.

A case is one pass of a controller, a router or an offline what-if study
through the entry points of ``paper_2408_05235_amd.api``: a whole step
(project, predict, select), the paper's binary search, admission of new
queries, the model on arbitrary rows, the step through the compiled lattice,
or the projection under length errors.  Board, request and model sizes are
those of ``paper_2408_05235_amd.configs`` (or lie between them); values follow
the same distributions, drawn here with torch on the GPU so that a case's
inputs are ready quickly.

Fields of a case: ``kind`` (the pass), ``S`` scenarios, ``H`` future
iterations, ``F`` candidate frequencies, ``R`` requests in flight per
scenario, ``queued`` requests waiting at iteration 0, ``rate`` arrivals per
iteration (0 = none), ``prompt`` / ``length`` (largest prompt and remaining
length; lengths are log-normal where there are arrivals), ``N`` tokens per KV
block, ``cap_kv`` blocks, ``cap_batch`` (0 = none), the model's ``T`` trees of
depth ``d`` over ``nf`` features with KV and batch ranges ``cap_kv`` and
``bmax``, and ``rows`` for the pass on arbitrary rows.
"""
import math

import numpy as np
import torch

from paper_2408_05235_amd import api


def _case(name, kind, **kw):
    c = dict(name=name, kind=kind, S=1, H=512, F=17, R=64, queued=0, rate=0.0, prompt=1024, length=512, N=16,
             cap_kv=8192, cap_batch=0, T=100, d=6, nf=3, bmax=256, rows=0)
    c.update(kw)
    return c


def listed():
    return [
        # One serving engine's own controller: its board, 17 clock steps, the
        # small model.  Called at every iteration of the engine, so the time
        # of this call is what the controller adds to serving.
        _case("step_one_board", "step"),
        # The same controller as the paper states it (binary search), on a
        # longer board with 64 clock steps and the 500-tree model.
        _case("search_one_board", "search", S=1, R=256, H=2048, F=64, prompt=4096, length=2048, cap_kv=65536, T=500,
              d=8),
        # A router asks eight engines of different sizes whether they take one
        # more query: the 4-feature model at the highest clock.
        _case("admit_eight_boards", "admit", S=8, R=128, H=1024, F=64, length=1024, cap_kv=65536, T=2000, d=10, nf=4,
              bmax=128),
        # A small fleet with sizes off every tile: 37 boards, 777 iterations,
        # 23 clock steps, 24-token blocks.
        _case("step_ragged_fleet", "step", S=37, R=91, H=777, F=23, N=24, prompt=2000, length=900, cap_kv=20000,
              T=250, d=7, bmax=192),
        # What-if study over 1024 boards of 256 requests.
        _case("step_1024_boards", "step", S=1024, R=256, H=2048, F=64, prompt=4096, length=2048, cap_kv=65536, T=500,
              d=8),
        # Long contexts, 256 requests waiting behind a batch cap of 256.
        _case("step_long_context", "step", S=256, R=256, queued=256, H=4096, F=32, prompt=32768, length=4096,
              cap_kv=1 << 20, cap_batch=256, T=300, d=8),
        # The model-bound study: 4096 boards, 2000 trees of depth 10 over four
        # features (engine sizes 1, 2, 4, 8).  The largest listed case.
        _case("step_4096_boards_large_model", "step", S=4096, R=128, H=1024, F=64, length=1024, cap_kv=65536, T=2000,
              d=10, nf=4, bmax=128),
        # The binary search over the 1024 boards.
        _case("search_1024_boards", "search", S=1024, R=256, H=2048, F=64, prompt=4096, length=2048, cap_kv=65536,
              T=500, d=8),
        # Admission what-ifs for boards under Poisson arrivals: thousands of
        # queued and arriving requests per board go through the FIFO.
        _case("admit_arrivals", "admit", S=8192, R=256, rate=8.0, H=2048, F=48, prompt=2048, length=8192,
              cap_kv=131072, T=800, d=8, bmax=2048),
        # The model on a caller's own feature rows (an odd number of them).
        _case("rows_million", "rows", rows=1000003, F=64, cap_kv=65536, T=500, d=8),
        # The step through the model compiled to its lattice.
        _case("lattice_1024_boards", "lattice", S=1024),
        # The scoreboard under length errors, then its projection: boards
        # whose KV capacity binds under arrivals.
        _case("project_arrivals", "project", S=4096, R=256, rate=8.0, H=2048, prompt=2048, length=8192,
              cap_kv=131072),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "step", "step", "search", "search", "admit", "admit", "rows", "lattice", "project"])
    c = _case("", kind)
    del c["name"]
    nf = rng.choice([3, 3, 4])
    c.update(H=logint(200, 4096), F=rng.choice([rng.randint(9, 96), 17, 32, 48, 64]), R=logint(16, 256),
             N=rng.choice([16, 16, 16, 8, 32, 24]), prompt=logint(512, 8192), nf=nf, T=logint(60, 2000),
             d=rng.randint(5, 10), bmax=rng.choice([128, 256, 512]))
    c["cap_kv"] = rng.choice([8192, 32768, 65536, 131072])
    c["length"] = max(64, int(c["H"] * rng.uniform(0.5, 1.2)))
    board = rng.choice(["inflight", "inflight", "queued", "arrivals"])
    if kind == "project":
        board = rng.choice(["queued", "arrivals"])
    if kind in ("lattice", "rows"):
        board = "inflight"
    per = c["R"]
    if board == "queued":
        c["queued"] = logint(16, 256)
        c["cap_batch"] = rng.choice([0, c["R"], c["R"] + 16])
        per += c["queued"]
    elif board == "arrivals":
        c["rate"] = rng.uniform(1.0, 8.0)
        c["length"] = 8192
        c["bmax"] = 2048
        per += int(c["rate"] * c["H"])
    rows = {"step": c["F"], "search": math.ceil(math.log2(c["F"])) + 1, "admit": 1}.get(kind, 1) * c["H"]
    most = min(4096, int(3e7 / per) + 1, int(1.5e8 / rows) + 1)
    if kind in ("step", "search", "admit"):
        most = min(most, int(1e11 / (rows * c["T"])) + 1)
    if kind == "lattice":
        c.update(F=rng.choice([17, 31, 64]), cap_kv=8192, bmax=128, R=min(c["R"], 128), prompt=512, T=min(c["T"], 200),
                 d=min(c["d"], 7), nf=3)
        most = min(2048, int(1e8 / (c["F"] * c["H"])) + 1)
    c["S"] = logint(1, max(1, most))
    if kind == "rows":
        c["rows"] = logint(1000, 4000000)
        c["T"] = min(c["T"], int(4e12 / (c["rows"] * c["d"])) + 1)
    return c


# ------------------------------------------------------------------ inputs


def _lengths(g, case, shape):
    if case["rate"] > 0:    # tens to hundreds of tokens with a long tail
        z = torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
        return torch.exp(5.0 + 1.2 * z).round().clamp(1, case["length"]).to(torch.int32)
    return torch.randint(1, case["length"] + 1, shape, generator=g, device="cuda", dtype=torch.int32)


def _prompts(g, case, shape):
    if case["prompt"] >= 16384:     # long contexts: log-normal
        z = torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)
        return torch.exp(8.0 + z).round().clamp(1, case["prompt"]).to(torch.int32)
    return torch.randint(16, case["prompt"] + 1, shape, generator=g, device="cuda", dtype=torch.int32)


def _frequencies(F):
    k = torch.arange(F, dtype=torch.int64, device="cuda")
    return (1000 + (k * 1000) // max(1, F - 1)).to(torch.float32)


def _boards(case, g):
    """Scoreboards on the GPU, laid out as ``api.upload`` lays them out."""
    S, H, R, Q = case["S"], case["H"], case["R"], case["queued"]
    dev = "cuda"
    n_arr = torch.zeros(S, dtype=torch.int64, device=dev)
    counts = None
    if case["rate"] > 0:
        # Poisson arrivals, each board at a rate of its own, given their total
        rate = 0.0625 + 0.9375 * torch.rand(S, generator=g, device=dev, dtype=torch.float64)
        edge = torch.cumsum(rate, 0)
        n = int(0.53125 * case["rate"] * H * S)
        at = torch.rand(n, generator=g, device=dev, dtype=torch.float64) * edge[-1]
        s = torch.searchsorted(edge, at).clamp(max=S - 1)
        j = torch.randint(0, H, (n,), generator=g, device=dev)
        counts = torch.bincount(s * H + j, minlength=S * H).reshape(S, H)
        n_arr = counts.sum(1)
    off = torch.zeros(S + 1, dtype=torch.int64, device=dev)
    off[1:] = torch.cumsum(n_arr + (R + Q), 0)
    total = int(off[-1])
    arrival = torch.full((total,), -1, dtype=torch.int32, device=dev)
    within = torch.arange(total, device=dev) - torch.repeat_interleave(off[:-1], n_arr + (R + Q), output_size=total)
    inflight = within < R
    arrival[(within >= R) & (within < R + Q)] = 0
    if counts is not None:
        its = torch.arange(H, dtype=torch.int32, device=dev).repeat(S)
        arrival[within >= R + Q] = torch.repeat_interleave(its, counts.reshape(-1), output_size=int(n_arr.sum()))
    prompt = _prompts(g, case, (total,))
    remaining = _lengths(g, case, (total,))
    generated = torch.where(inflight, torch.randint(0, 257, (total,), generator=g, device=dev, dtype=torch.int32), 0)
    del within
    # per-token SLOs of 10 to 50 ms; requests in flight must finish at that
    # pace, the others carry no deadline yet
    slo = torch.randint(10000, 50001, (S,), generator=g, device=dev, dtype=torch.int64) * 1000
    which = torch.repeat_interleave(torch.arange(S, device=dev), n_arr + (R + Q), output_size=total)
    deadline = torch.where(inflight, slo[which] * remaining, -1)
    lost = torch.zeros(total, dtype=torch.uint8, device=dev)
    has = torch.rand(S, generator=g, device=dev) < 1.0 / 64
    pick = torch.randint(0, R, (S,), generator=g, device=dev)
    lost[(off[:-1] + pick)[has]] = 1
    engine = None
    if case["nf"] == 4:
        engine = torch.tensor([1.0, 2.0, 4.0, 8.0], device=dev)[torch.randint(0, 4, (S,), generator=g, device=dev)]
    full = lambda v: torch.full((S,), v, dtype=torch.int32, device=dev)  # noqa: E731
    return dict(n_scenarios=S, horizon=H, block_tokens=case["N"], n_features=case["nf"], req_offset=off,
                prompt=prompt, generated=generated, remaining=remaining, arrival=arrival, deadline_ns=deadline,
                lost=lost, kv_capacity=full(case["cap_kv"]),
                batch_cap=full(case["cap_batch"]) if case["cap_batch"] else None, tbt_slo_ns=slo,
                freqs_mhz=_frequencies(case["F"]), engine_size=engine)


def _model(case, g):
    """A gradient-boosted ensemble whose leaves follow a smooth surface of
    iterations per second (slower at low clocks, large batches and full KV
    caches); one threshold in ten lies on a value that the inputs take."""
    T, d, nf = case["T"], case["d"], case["nf"]
    dev, f64 = "cuda", torch.float64
    top = torch.tensor([2000.0, float(case["cap_kv"]), float(case["bmax"]), 8.0][:nf], dtype=f64, device=dev)
    low = torch.tensor([1000.0, 0.0, 0.0, 1.0][:nf], dtype=f64, device=dev)
    lo, hi = low.repeat(T, 1, 1), top.repeat(T, 1, 1)
    freqs = _frequencies(case["F"]).to(f64)
    feature, threshold = [], []
    for level in range(d):
        w = 1 << level
        ft = torch.randint(0, nf, (T, w), generator=g, device=dev)
        a, b = lo.gather(2, ft[..., None])[..., 0], hi.gather(2, ft[..., None])[..., 0]
        th = a + (b - a) * torch.rand((T, w), generator=g, device=dev, dtype=f64)
        snap = torch.rand((T, w), generator=g, device=dev) < 0.1
        near = freqs[torch.searchsorted(freqs, th.clamp(1000.0, 2000.0)).clamp(max=len(freqs) - 1)]
        th = torch.where(snap, torch.where(ft == 0, near, th.round()), th).to(torch.float32)
        feature.append(ft.to(torch.uint8))
        threshold.append(th)
        hit = torch.nn.functional.one_hot(ft, nf).bool()
        t3 = th.to(f64)[..., None]
        lo = torch.stack([lo, torch.where(hit, t3, lo)], 2).reshape(T, 2 * w, nf)
        hi = torch.stack([torch.where(hit, t3, hi), hi], 2).reshape(T, 2 * w, nf)
    mid = 0.5 * (lo + hi)
    noise = torch.randn((T, 1 << d), generator=g, device=dev, dtype=f64)
    if nf == 4:
        leaf = 0.1 * noise
    else:
        tbt = 12.0 * (2000.0 / mid[..., 0]) ** 0.8 * (1.0 + 0.5 * mid[..., 2] / case["bmax"]
                                                      + 0.5 * mid[..., 1] / case["cap_kv"])
        leaf = (1000.0 / tbt - 40.0) / T + 0.01 * noise
    cat = lambda parts: torch.cat(parts, 1).cpu().numpy() if parts else np.zeros((T, 0))  # noqa: E731
    return dict(n_trees=T, depth=d, n_features=nf, base_score=40.0, feature=cat(feature), threshold=cat(threshold),
                leaf=leaf.to(torch.float32).cpu().numpy())


def _inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(0x74686C + 1000003 * int(seed))
    return g


def _rows(case, g):
    top = torch.tensor([1000.0, float(case["cap_kv"]), float(case["bmax"]), 7.0][: case["nf"]], device="cuda")
    x = (torch.rand((case["rows"], case["nf"]), generator=g, device="cuda") * top).round()
    x[:, 0] += 1000.0
    if case["nf"] == 4:
        x[:, 3] = 2.0 ** torch.randint(0, 4, (case["rows"],), generator=g, device="cuda").to(torch.float32)
    return x


def prepare(case, seed):
    g = _inputs(case, seed)
    kind = case["kind"]
    state = dict(case=case)
    if kind != "project":
        state["forest"] = api.Forest.from_dict(_model(case, g))
    if kind == "rows":
        state["rows"] = _rows(case, g)
        state["out"] = torch.empty(case["rows"], dtype=torch.float32, device="cuda")
        return state
    d = state["d"] = _boards(case, g)
    S, H, dev = case["S"], case["H"], "cuda"
    i32 = torch.int32
    if kind in ("step", "search", "lattice"):
        state["ctl"] = api.Controller(d, state["forest"])
    if kind == "lattice":
        state["lat"] = api.Lattice(state["forest"], d["freqs_mhz"], case["cap_kv"], case["bmax"])
    if kind == "search":
        state["out"] = dict(ips_work=torch.zeros((S, H), device=dev), search_work=torch.zeros((3, S), dtype=i32, device=dev),
                            freq_idx=torch.zeros(S, dtype=i32, device=dev), status=torch.zeros(S, dtype=i32, device=dev))
    if kind in ("admit", "project"):
        state["out"] = dict(batch=torch.empty((S, H), dtype=i32, device=dev), kv=torch.empty((S, H), dtype=i32, device=dev),
                            deadline_at=torch.empty((S, H), dtype=torch.int64, device=dev),
                            n_iters=torch.empty(S, dtype=i32, device=dev), flags=torch.empty(S, dtype=i32, device=dev))
    if kind == "admit":
        state["out"].update(ips=torch.empty((S, H), device=dev), decision=torch.empty(S, dtype=i32, device=dev))
        state["cand_prompt"] = _prompts(g, case, (S,))
        state["cand_len"] = _lengths(g, case, (S,))
        state["cand_deadline"] = d["tbt_slo_ns"] * state["cand_len"]
        state["fmax"] = float(d["freqs_mhz"][-1])
    if kind == "project":
        # predicted total lengths, inflated by the predictor's error (5 to 25%)
        state["pred"] = (d["generated"] + d["remaining"]).to(i32)
        state["num"] = torch.randint(105, 126, (S,), generator=g, device=dev, dtype=i32)
        state["den"] = torch.full((S,), 100, dtype=i32, device=dev)
        state["most"] = torch.full((S,), 8192, dtype=i32, device=dev)
        state["remaining"] = torch.empty_like(d["remaining"])
    return state


def run(state):
    kind, d = state["case"]["kind"], state.get("d")
    if kind == "rows":
        return state["forest"].tl_forest_predict(state["rows"], state["out"])
    if kind == "step":
        ctl = state["ctl"]
        idx, status = ctl.step()
        return dict(ctl.buf, ips=ctl.ips, freq_idx=idx, status=status)
    if kind == "search":
        ctl, out = state["ctl"], state["out"]
        p = ctl.project()
        idx, status = api.tl_select_freq_binary(state["forest"], d["freqs_mhz"], p["kv"], p["batch"], p["deadline_at"],
                                                p["n_iters"], d["tbt_slo_ns"], p["flags"], d["engine_size"], out)
        return dict(p, ips=out["ips_work"], freq_idx=idx, status=status)
    if kind == "lattice":
        ctl = state["ctl"]
        p = ctl.project()
        ips = state["lat"].tl_lattice_predict_grid(p["kv"], p["batch"], d["engine_size"], ctl.ips)
        idx, status = ctl.select()
        return dict(p, ips=ips, freq_idx=idx, status=status)
    if kind == "admit":
        return api.tl_admit(state["forest"], state["fmax"], d["tbt_slo_ns"], state["cand_prompt"], state["cand_len"],
                            d["req_offset"], d["prompt"], d["generated"], d["remaining"], d["arrival"],
                            d["kv_capacity"], d["horizon"], d["block_tokens"], d["deadline_ns"], d["lost"],
                            d["batch_cap"], d["engine_size"], state["cand_deadline"], state["out"])
    rem = api.tl_adjust_lengths(d["req_offset"], d["generated"], state["pred"], state["num"], state["den"],
                                state["most"], state["remaining"])
    p = api.tl_project(d["req_offset"], d["prompt"], d["generated"], rem, d["arrival"], d["kv_capacity"], d["horizon"],
                       d["block_tokens"], d["deadline_ns"], d["lost"], d["batch_cap"], want_rows=False, out=state["out"])
    return dict(p, remaining=rem)


# ------------------------------------------------------- cost and tolerance


def work(case):
    """Requests read once (25 bytes each), curves written (16 bytes per
    iteration), predictions written; one fp32 addition per (row, tree)."""
    S, H, F, T = case["S"], case["H"], case["F"], case["T"]
    model = T * (1 << case["d"]) * 12
    if case["kind"] == "rows":
        return {"bytes": case["rows"] * 4 * (case["nf"] + 1) + model, "flops": case["rows"] * T}
    per = case["R"] + case["queued"] + (0.53125 * case["rate"] * H)
    board = S * per * 25 + S * H * 16 + S * 32
    if case["kind"] == "step":
        return {"bytes": board + S * F * H * 4 + model, "flops": S * F * H * T}
    if case["kind"] == "search":
        return {"bytes": board + S * H * 4 + model, "flops": S * H * T * math.ceil(math.log2(max(2, F)))}
    if case["kind"] == "admit":
        return {"bytes": board + S * H * 4 + model, "flops": S * H * T}
    if case["kind"] == "lattice":
        return {"bytes": board + S * F * H * 8, "flops": S * H * per}
    return {"bytes": board + S * per * 12, "flops": S * per}


def tolerance(case):
    """Curves, flags, decisions and indices are whole numbers, and the
    library's interface fixes every fp32 sum: the base, then the trees in
    order, each addition rounded to nearest (two runs of the library, and the
    library and its oracle, give the same bits)."""
    return "exact"


def _curves(case, d, cand=None):
    """KV blocks and batch size per iteration of boards without a queue."""
    S, H, N, R = case["S"], case["H"], case["N"], case["R"]
    c = (d["prompt"] + d["generated"]).to(torch.int64).reshape(S, R)
    r = d["remaining"].to(torch.int64).reshape(S, R)
    if cand is not None:
        c = torch.cat([c, cand[0].to(torch.int64)[:, None]], 1)
        r = torch.cat([r, cand[1].to(torch.int64)[:, None]], 1)
    kv, batch = [], []
    for j in range(H):
        on = r > j
        kv.append((((c + j + N - 1) // N) * on).sum(1))
        batch.append(on.sum(1))
    return torch.stack(kv, 1), torch.stack(batch, 1)


def _evaluate(model, x):
    """The ensemble on rows x in float64."""
    T, d = model["n_trees"], model["depth"]
    ft = torch.from_numpy(model["feature"].astype(np.int64)).cuda()
    th = torch.from_numpy(model["threshold"]).cuda()
    leaf = torch.from_numpy(model["leaf"]).cuda().to(torch.float64)
    n_int = (1 << d) - 1
    out = torch.empty(x.shape[0], dtype=torch.float64, device="cuda")
    step = 1 << 20
    for a in range(0, x.shape[0], step):
        xs = x[a:a + step]
        acc = torch.full((xs.shape[0],), float(model["base_score"]), dtype=torch.float64, device="cuda")
        for t in range(T):
            k = torch.zeros(xs.shape[0], dtype=torch.int64, device="cuda")
            for _ in range(d):
                v = xs.gather(1, ft[t][k][:, None])[:, 0]
                k = 2 * k + 2 - (v < th[t][k]).to(torch.int64)
            acc += leaf[t][k - n_int]
        out[a:a + step] = acc
    return out


def exact(case, seed):
    kind = case["kind"]
    n = {"rows": case["rows"], "step": case["S"] * case["F"] * case["H"], "lattice": case["S"] * case["F"] * case["H"],
         "admit": case["S"] * case["H"]}.get(kind)
    if n is None or case["queued"] or case["rate"] > 0 or n * case["T"] * case["d"] > 2e10 or \
            case["T"] * case["d"] * (n // (1 << 20) + 1) > 60000:
        return None
    g = _inputs(case, seed)
    model = _model(case, g)
    if kind == "rows":
        return _evaluate(model, _rows(case, g))
    d = _boards(case, g)
    S, H = case["S"], case["H"]
    freqs = d["freqs_mhz"]
    cand = None
    if kind == "admit":
        cand = (_prompts(g, case, (S,)), _lengths(g, case, (S,)))
        freqs = freqs[-1:]
    kv, batch = _curves(case, d, cand)
    F = freqs.numel()
    cols = [freqs[None, :, None].expand(S, F, H), kv[:, None, :].expand(S, F, H).to(torch.float32),
            batch[:, None, :].expand(S, F, H).to(torch.float32)]
    if case["nf"] == 4:
        cols.append(d["engine_size"][:, None, None].expand(S, F, H))
    ips = _evaluate(model, torch.stack([c.reshape(-1) for c in cols], 1)).reshape(S, F, H)
    if kind == "admit":
        ips = ips.reshape(S, H)
    names = ["batch", "kv", "deadline_at", "n_iters", "flags", "ips"]
    names += ["decision"] if kind == "admit" else ["freq_idx", "status"]
    return {k: ips if k == "ips" else None for k in names}
