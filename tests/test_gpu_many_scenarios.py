"""More scenarios than workgroups of 256 threads fit in one launch (2^24):
projection, prediction, selection, binary search and admission on short boards,
a block of different ones repeated, against the oracle on the block."""
import numpy as np
import pytest

import oracle
from paper_2408_05235_amd import synth
from test_gpu_parity import random_forest

pytestmark = pytest.mark.gpu

BLOCK, H, F = 37, 2, 2
S = BLOCK * ((1 << 24) // BLOCK + 1)      # a few more than 2^24


def _block(rng):
    n = BLOCK * 2
    return dict(n_scenarios=BLOCK, horizon=H, block_tokens=16, req_offset=np.arange(BLOCK + 1, dtype=np.int64) * 2,
                prompt=rng.integers(1, 300, n).astype(np.int32), generated=rng.integers(0, 50, n).astype(np.int32),
                remaining=rng.integers(1, 4, n).astype(np.int32),
                arrival=np.tile(np.array([-1, 0], np.int32), BLOCK),
                deadline_ns=rng.integers(1, 10 ** 8, n).astype(np.uint64),
                lost=(rng.random(n) < 0.05).astype(np.uint8),
                kv_capacity=rng.integers(10, 40, BLOCK).astype(np.int32), batch_cap=None)


def _same(got, exp, name):
    """Every scenario's part of `got` [S, ...] against the block's."""
    import torch
    e = torch.from_numpy(np.ascontiguousarray(exp).view(f"i{exp.dtype.itemsize}")).cuda()
    g = got.view(e.dtype).reshape((S // BLOCK,) + tuple(e.shape))
    assert bool((g == e).all()), name


def test_more_than_2_24_scenarios(gpu):
    import torch
    from paper_2408_05235_amd import api
    rng = np.random.default_rng(52)
    inp = _block(rng)
    fd = random_forest(rng, 3, 3, 3, kvmax=60, bmax=4)
    freqs = synth.frequency_grid(F)
    slo = rng.integers(10, 60, BLOCK).astype(np.uint64) * 10 ** 6
    cand_p = rng.integers(1, 200, BLOCK).astype(np.int32)
    cand_l = rng.integers(1, 4, BLOCK).astype(np.int32)
    cand_d = rng.integers(1, 10 ** 8, BLOCK).astype(np.uint64)
    rep = S // BLOCK
    t = lambda a: torch.from_numpy(a.view(np.int64) if a.dtype == np.uint64 else a).cuda().repeat(rep)
    off = torch.arange(S + 1, device="cuda", dtype=torch.int64) * 2
    d = {k: t(inp[k]) for k in ("prompt", "generated", "remaining", "arrival", "deadline_ns", "lost", "kv_capacity")}
    args = (off, d["prompt"], d["generated"], d["remaining"], d["arrival"], d["kv_capacity"], H, 16,
            d["deadline_ns"], d["lost"], None)
    forest = api.Forest.from_dict(fd)
    dslo, dfr = t(slo), torch.from_numpy(freqs).cuda()

    exp = oracle.project(inp)
    p = api.tl_project(*args, want_rows=False)
    for k in ("batch", "kv", "deadline_at", "n_iters", "flags"):
        _same(p[k], exp[k], k)
    ips = oracle.forest_predict(fd, oracle.rows(freqs, exp["batch"], exp["kv"], None, 3))
    got = forest.tl_forest_predict_grid(dfr, p["kv"], p["batch"])
    _same(got, ips, "ips")
    i, s = oracle.select(ips, exp["deadline_at"], exp["n_iters"], slo, exp["flags"])
    gi, gs = api.tl_select_freq(got, p["deadline_at"], p["n_iters"], dslo, p["flags"])
    _same(gi, i, "freq_idx")
    _same(gs, s, "status")
    bi, bs = oracle.select_binary(ips, exp["deadline_at"], exp["n_iters"], slo, exp["flags"])
    gi, gs = api.tl_select_freq_binary(forest, dfr, p["kv"], p["batch"], p["deadline_at"], p["n_iters"], dslo,
                                       p["flags"])
    _same(gi, bi, "binary freq_idx")
    _same(gs, bs, "binary status")
    # the model as a table, and the lengths
    lat = api.Lattice(forest, dfr, 60, 4)
    _same(lat.tl_lattice_predict_grid(p["kv"], p["batch"]), ips, "lattice")
    gi, _ = api.tl_select_freq_binary(forest, dfr, p["kv"], p["batch"], p["deadline_at"], p["n_iters"], dslo,
                                      p["flags"], lattice=lat)
    _same(gi, bi, "binary freq_idx with the lattice")
    lat.close()
    ones = np.full(BLOCK, 1, np.uint32)
    exp_len = oracle.adjust_lengths(inp["req_offset"], inp["generated"], inp["remaining"] * 30, ones * 11, ones * 10,
                                    np.full(BLOCK, 70, np.int32))
    got_len = api.tl_adjust_lengths(off, d["generated"], d["remaining"] * 30, t(ones.view(np.int32) * 11),
                                    t(ones.view(np.int32) * 10), t(np.full(BLOCK, 70, np.int32)))
    _same(got_len, exp_len, "lengths")
    del got, p
    a = oracle.admit(dict(inp, tbt_slo_ns=slo), cand_p, cand_l, cand_d, float(freqs[-1]), fd)
    g = api.tl_admit(forest, float(freqs[-1]), dslo, t(cand_p), t(cand_l), *args, None, t(cand_d))
    for k in ("batch", "kv", "deadline_at", "n_iters", "flags", "decision"):
        _same(g[k], a[k], "admit " + k)
    forest.close()
