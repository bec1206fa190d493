"""The staged forest kernels at the edges of their tiles and rank groups,
against the oracle, bit for bit: horizons around the 32-row chunks and the
64-row work-order entries, frequency counts around a wavefront, odd numbers of
trees, the deepest records, and a forest with more thresholds per feature than
one rank group holds (grid, search probes and arbitrary rows)."""
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
