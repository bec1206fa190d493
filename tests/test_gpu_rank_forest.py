"""The staged forest kernels at the edges of their tiles and rank groups,
against the oracle, bit for bit: horizons around the 32-row chunks and the
64-row work-order entries, frequency counts around a wavefront, odd numbers of
trees, the deepest records, a forest with more thresholds per feature than
one rank group holds (grid, search probes and arbitrary rows), and sizes on
each side of the rules that choose a kernel for few, some and many rows."""
import numpy as np
import pytest

import oracle
from paper_2408_05235_amd import synth
from test_gpu_parity import random_curves, random_forest

pytestmark = pytest.mark.gpu


def _dev(a, dt):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dt)).cuda()


def _grid(fd, freqs, kv, bs, eng):
    from paper_2408_05235_amd import api
    f = api.Forest.from_dict(fd)
    got = f.tl_forest_predict_grid(_dev(freqs, np.float32), _dev(kv, np.int32), _dev(bs, np.int32),
                                   None if eng is None else _dev(eng, np.float32)).cpu().numpy()
    x = oracle.rows(freqs, bs, kv, eng, fd["n_features"])
    exp = oracle.forest_predict(fd, x).reshape(got.shape)
    rows = f.tl_forest_predict(_dev(np.asarray(x, np.float32).reshape(-1, fd["n_features"]), np.float32)).cpu().numpy()
    f.close()
    assert np.array_equal(got, exp)
    assert np.array_equal(rows.reshape(got.shape), exp)


@pytest.mark.parametrize("S,H,F,T,d,nf", [
    (1, 1, 1, 1, 0, 3), (3, 31, 17, 3, 1, 4), (2, 32, 64, 2, 8, 3), (5, 33, 65, 7, 7, 4), (40, 63, 23, 9, 5, 3),
    (7, 64, 48, 5, 11, 4), (2, 65, 128, 21, 9, 3), (33, 97, 33, 1, 10, 4), (70, 130, 96, 11, 6, 3),
])
def test_tile_edges(S, H, F, T, d, nf):
    rng = np.random.default_rng(S * 1000 + H)
    fd = random_forest(rng, T, d, nf, kvmax=3000, bmax=200)
    kv, bs = random_curves(rng, S, H, kvmax=3000, bmax=200)
    eng = rng.choice([1.0, 2.0, 4.0, 8.0], S).astype(np.float32) if nf == 4 else None
    _grid(fd, synth.frequency_grid(F), kv, bs, eng)


@pytest.mark.parametrize("nf", [3, 4])
def test_several_rank_groups(nf):
    rng = np.random.default_rng(nf)
    T, d = 320, 10                       # 320 x 1023 / nf > 65534 thresholds per feature
    fd = synth.make_forest(rng, T, d, nf, "normal", 40.0, 60000, 200, synth.frequency_grid(20))
    S, H, F = 2, 70, 20
    kv, bs = random_curves(rng, S, H, kvmax=60000, bmax=200)
    eng = np.array([2.0, 8.0], np.float32) if nf == 4 else None
    _grid(fd, synth.frequency_grid(F), kv, bs, eng)


@pytest.mark.parametrize("H,S", [(512, 8192), (1024, 4096)])
def test_several_rank_groups_along_the_horizon(H, S):
    """The leaf-reuse column kernel (8 and 16 rows a lane): one candidate
    frequency leaves M at it in the search's work array."""
    import torch
    from paper_2408_05235_amd import api
    rng = np.random.default_rng(H)
    nf, T, d = 4, 280, 10
    freqs = np.array([1400.0], np.float32)
    fd = synth.make_forest(rng, T, d, nf, "normal", 40.0, 60000, 200, synth.frequency_grid(20))
    kv, bs = random_curves(rng, S, H, kvmax=60000, bmax=200)
    eng = rng.choice([1.0, 2.0, 4.0, 8.0], S).astype(np.float32)
    f = api.Forest.from_dict(fd)
    work = dict(ips_work=torch.zeros((S, H), device="cuda"))
    full = lambda v, dt: torch.full((S,), v, dtype=dt, device="cuda")
    api.tl_select_freq_binary(f, _dev(freqs, np.float32), _dev(kv, np.int32), _dev(bs, np.int32),
                              torch.full((S, H), -1, dtype=torch.int64, device="cuda"), full(H, torch.int32),
                              full(30_000_000, torch.int64), None, _dev(eng, np.float32), work)
    got = work["ips_work"].cpu().numpy()
    f.close()
    pick = np.array([0, 1, S // 2, S - 1])
    exp = oracle.forest_predict(fd, oracle.rows(freqs, bs[pick], kv[pick], eng[pick], nf)).reshape(len(pick), H)
    assert np.array_equal(got[pick], exp)


# too few trees to run as a call with few rows: 8, 16 or 32 grid rows a
# wavefront (the last also with a work order), and one or two column rows a lane
@pytest.mark.parametrize("S,F,H", [(5, 70, 190), (40, 70, 190), (250, 9, 190), (500, 5, 190), (1500, 3, 190)])
def test_grid_kernel_choice(S, F, H):
    rng = np.random.default_rng(S)
    fd = random_forest(rng, 3, 11, 4, kvmax=3000, bmax=200)
    kv, bs = random_curves(rng, S, H, kvmax=3000, bmax=200)
    _grid(fd, synth.frequency_grid(F), kv, bs, rng.choice([1.0, 2.0, 4.0, 8.0], S).astype(np.float32))


@pytest.mark.parametrize("captured", [False, True])
@pytest.mark.parametrize("S,H", [(3, 65), (1000, 190), (4100, 100)])
def test_column_kernel_choice(S, H, captured):
    """One candidate frequency leaves M at it in the search's work array;
    scenarios flagged lost are left alone.  Captured into a graph the call has
    no scratch and takes the column kernel whatever the size."""
    import torch
    from paper_2408_05235_amd import api
    rng = np.random.default_rng(H)
    fd = random_forest(rng, 5, 11, 3, kvmax=3000, bmax=200)
    kv, bs = random_curves(rng, S, H, kvmax=3000, bmax=200)
    freqs = np.array([1400.0], np.float32)
    lost = rng.random(S) < 0.2
    f = api.Forest.from_dict(fd)
    out = dict(ips_work=torch.full((S, H), -1.0, device="cuda"), search_work=torch.zeros((3, S), dtype=torch.int32, device="cuda"),
               freq_idx=torch.zeros(S, dtype=torch.int32, device="cuda"), status=torch.zeros(S, dtype=torch.int32, device="cuda"))
    full = lambda v, dt: torch.full((S,), v, dtype=dt, device="cuda")
    args = (f, _dev(freqs, np.float32), _dev(kv, np.int32), _dev(bs, np.int32),
            torch.full((S, H), -1, dtype=torch.int64, device="cuda"), full(H, torch.int32),
            full(30_000_000, torch.int64), _dev(lost * 2, np.int32), None, out)
    if captured:
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            api.tl_select_freq_binary(*args)
        g.replay()
        torch.cuda.synchronize()
    else:
        api.tl_select_freq_binary(*args)
    got = out["ips_work"].cpu().numpy()
    exp = oracle.forest_predict(fd, oracle.rows(freqs, bs, kv, None, 3)).reshape(S, H)
    exp[lost] = -1.0
    assert np.array_equal(got, exp)
    f.close()


@pytest.mark.parametrize("n", [1, 63, 1025, 200_001, 530_001])
def test_rows_kernel_choice(n):
    import torch
    from paper_2408_05235_amd import api
    rng = np.random.default_rng(n)
    fd = random_forest(rng, 9, 11, 4, kvmax=3000, bmax=200)
    x = np.stack([rng.integers(900, 2100, n), rng.integers(-5, 3500, n), rng.random(n) * 220,
                  rng.choice([1.0, 2.0, 4.0, 8.0], n)], 1).astype(np.float32)
    x[rng.random(n) < 0.01, 1] = np.nan
    f = api.Forest.from_dict(fd)
    got = f.tl_forest_predict(_dev(x, np.float32)).cpu().numpy()
    f.close()
    assert np.array_equal(got, oracle.forest_predict(fd, x).reshape(-1))


@pytest.mark.parametrize("T", [255, 256, 257, 4000])
def test_few_rows_many_trees(T):
    """Trees around one LDS segment of the sum, and several slices of rows."""
    rng = np.random.default_rng(T)
    fd = random_forest(rng, T, 2 if T > 1000 else 5, 3, kvmax=3000, bmax=200)
    S, F, H = (6, 20, 75) if T > 1000 else (2, 9, 77)
    kv, bs = random_curves(rng, S, H, kvmax=3000, bmax=200)
    _grid(fd, synth.frequency_grid(F), kv, bs, None)


@pytest.mark.parametrize("S,F,H,T,d,nf", [
    (1, 17, 16, 21, 4, 3), (1, 17, 16, 22, 4, 3), (5, 70, 190, 12, 11, 4), (5, 70, 190, 13, 11, 4), (1, 1, 1, 101, 1, 3),
    (2, 30, 500, 300, 1, 4), (2, 31, 500, 300, 1, 4),
])
def test_few_rows_choice(S, F, H, T, d, nf):
    """Calls on each side of the rule by rows and levels that gives calls with
    few rows two launches (the grid's rows as a caller's own as well)."""
    rng = np.random.default_rng(S * F + T)
    fd = random_forest(rng, T, d, nf, kvmax=3000, bmax=200)
    kv, bs = random_curves(rng, S, H, kvmax=3000, bmax=200)
    _grid(fd, synth.frequency_grid(F), kv, bs, rng.choice([1.0, 2.0, 4.0, 8.0], S).astype(np.float32) if nf == 4 else None)


@pytest.mark.parametrize("S,H,T", [(3, 65, 18), (3, 65, 19), (700, 190, 60), (1000, 190, 60), (1100, 1, 40)])
def test_few_column_rows_choice(S, H, T):
    """The same for one candidate frequency per scenario, some flagged lost."""
    import torch
    from paper_2408_05235_amd import api
    rng = np.random.default_rng(S)
    fd = random_forest(rng, T, 11, 3, kvmax=3000, bmax=200)
    kv, bs = random_curves(rng, S, H, kvmax=3000, bmax=200)
    lost = rng.random(S) < 0.2
    f = api.Forest.from_dict(fd)
    out = dict(ips_work=torch.full((S, H), -1.0, device="cuda"))
    full = lambda v, dt: torch.full((S,), v, dtype=dt, device="cuda")
    freqs = np.array([1400.0], np.float32)
    api.tl_select_freq_binary(f, _dev(freqs, np.float32), _dev(kv, np.int32), _dev(bs, np.int32),
                              torch.full((S, H), -1, dtype=torch.int64, device="cuda"), full(H, torch.int32),
                              full(30_000_000, torch.int64), _dev(lost * 2, np.int32), None, out)
    got = out["ips_work"].cpu().numpy()
    f.close()
    exp = oracle.forest_predict(fd, oracle.rows(freqs, bs, kv, None, 3)).reshape(S, H)
    exp[lost] = -1.0
    assert np.array_equal(got, exp)
