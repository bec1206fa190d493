"""Calls from several threads on the per-thread default stream, one handle for
a stream in every thread: predictions with few rows, small searches' grids and
ordered projections, which share scratch between calls, against the oracle."""
import ctypes
import threading

import numpy as np
import pytest

import oracle
from paper_2408_05235_amd import synth
from test_gpu_parity import assert_projection_equal, random_boards, random_curves, random_forest

pytestmark = pytest.mark.gpu

PER_THREAD = ctypes.c_void_p(2)      # hipStreamPerThread


def _on_threads(n, work):
    errors = []

    def run(k):
        import torch
        try:
            work(k)
            # the stream ends with its thread and is not waited for by a
            # synchronization of the device after that
            torch.cuda.ExternalStream(PER_THREAD.value).synchronize()
        except Exception as e:       # raised again below, on the test's own thread
            errors.append(e)

    threads = [threading.Thread(target=run, args=(k,)) for k in range(n)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
    assert not errors, errors
    assert not any(t.is_alive() for t in threads)


def test_predictions_on_per_thread_streams(gpu, monkeypatch):
    import torch
    from paper_2408_05235_amd import api
    rng = np.random.default_rng(48)
    n_threads, reps, n = 3, 40, 3000
    fd = random_forest(rng, 200, 8, 3)
    forest = api.Forest.from_dict(fd)
    freqs = synth.frequency_grid(64)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    cases = []
    for k in range(n_threads):
        kv, bs = random_curves(rng, 2, 40 + k)
        rows = np.asarray(oracle.rows(freqs, bs, kv, None, 3), np.float32)
        cases.append(dict(kv=t(kv), bs=t(bs), rows=t(rows.reshape(-1, 3)), exp=oracle.forest_predict(fd, rows),
                          by_rows=torch.full((reps, 2 * 64 * (40 + k)), -1.0, device="cuda"),
                          by_grid=torch.full((reps, 2, 64, 40 + k), -1.0, device="cuda")))
    dfr = t(freqs)
    torch.cuda.synchronize()
    monkeypatch.setattr(api, "_stream", lambda: PER_THREAD)

    def work(k):
        c = cases[k]
        for r in range(reps):
            forest.tl_forest_predict(c["rows"], c["by_rows"][r])
            forest.tl_forest_predict_grid(dfr, c["kv"], c["bs"], None, c["by_grid"][r])

    _on_threads(n_threads, work)
    torch.cuda.synchronize()
    for c in cases:
        for r in range(reps):
            assert np.array_equal(c["by_grid"][r].cpu().numpy(), c["exp"]), r
            assert np.array_equal(c["by_rows"][r].cpu().numpy().reshape(c["exp"].shape), c["exp"]), r
    forest.close()


def test_projections_on_per_thread_streams(gpu, monkeypatch):
    import torch
    from paper_2408_05235_amd import api
    rng = np.random.default_rng(49)
    n_threads, reps = 2, 8
    cases = []
    for k in range(n_threads):
        inp = random_boards(rng, 30 + 11 * k, 300, 16, rmax=3000, qfrac=0.6)
        inp["batch_cap"] = None
        assert int(inp["req_offset"][-1]) >= 1024 * inp["n_scenarios"]
        d = api.upload(dict(inp, tbt_slo_ns=np.zeros(inp["n_scenarios"], np.uint64),
                            freqs_mhz=np.zeros(1, np.float32), engine_size=None, n_features=3))
        cases.append((inp, d, []))
    torch.cuda.synchronize()
    monkeypatch.setattr(api, "_stream", lambda: PER_THREAD)

    def work(k):
        _, d, outs = cases[k]
        for _ in range(reps):
            outs.append(api.tl_project(d["req_offset"], d["prompt"], d["generated"], d["remaining"], d["arrival"],
                                       d["kv_capacity"], d["horizon"], d["block_tokens"], d["deadline_ns"], d["lost"],
                                       None, want_rows=False))

    _on_threads(n_threads, work)
    torch.cuda.synchronize()
    for inp, _, outs in cases:
        exp = oracle.project(inp)
        for o in outs:
            assert_projection_equal(dict(batch=o["batch"].cpu().numpy(), kv=o["kv"].cpu().numpy(),
                                         deadline_at=o["deadline_at"].cpu().numpy().view(np.uint64),
                                         n_iters=o["n_iters"].cpu().numpy(),
                                         flags=o["flags"].cpu().numpy().view(np.uint32)), exp)


def test_growing_calls_on_several_streams(gpu):
    """Row counts that grow from call to call, so that scratch is replaced while
    calls on other streams still use it."""
    import torch
    from paper_2408_05235_amd import api
    rng = np.random.default_rng(51)
    fd = random_forest(rng, 150, 7, 3)
    forest = api.Forest.from_dict(fd)
    x = np.stack([rng.integers(1000, 2001, 20000), rng.integers(0, 500, 20000), rng.integers(0, 60, 20000)],
                 1).astype(np.float32)
    exp = oracle.forest_predict(fd, x)
    dx = torch.from_numpy(x).cuda()
    streams = [torch.cuda.Stream() for _ in range(6)]
    outs = [torch.full((20000,), -1.0, device="cuda") for _ in range(60)]
    torch.cuda.synchronize()
    counts = [int(50 * 1.105 ** i) for i in range(60)]
    for i, n in enumerate(counts):
        with torch.cuda.stream(streams[i % 6]):
            forest.tl_forest_predict(dx[:n], outs[i][:n])
    torch.cuda.synchronize()
    for n, o in zip(counts, outs):
        assert np.array_equal(o[:n].cpu().numpy(), exp[:n]), n
    forest.close()
