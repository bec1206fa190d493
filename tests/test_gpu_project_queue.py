"""The projection's FIFO admission where its paths change, against the oracle:
queues around one and two chunks of 64 requests, capacities that never bind,
bind from the start or from some iteration on, unsorted arrivals, block sizes
with and without shifts, few and many boards (four wavefronts a board, or
one), and long queues without a batch cap."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import assert_projection_equal, gpu_project

pytestmark = pytest.mark.gpu


def _boards(seed, S, H, N, R, Q, cap_kv, cap_batch, unsorted):
    rng = np.random.default_rng(seed)
    n = R + Q
    total = S * n
    arrival = np.full((S, n), -1, np.int32)
    arrival[:, R:] = np.sort(rng.integers(0, H + H // 8, (S, Q)), axis=1)
    if unsorted:
        arrival[:, R:] = rng.permuted(arrival[:, R:], axis=1)
    arrival = arrival.reshape(-1)
    prompt = rng.integers(0, 600, total).astype(np.int32)
    prompt[rng.random(total) < 0.01] = -1                    # malformed entries
    remaining = np.clip(np.rint(rng.lognormal(4.0, 1.2, total)), 1, 4 * H).astype(np.int32)
    return dict(n_scenarios=S, horizon=H, block_tokens=N,
                req_offset=np.arange(S + 1, dtype=np.int64) * n, prompt=prompt,
                generated=np.where(arrival < 0, rng.integers(0, 100, total), 0).astype(np.int32),
                remaining=remaining, arrival=arrival,
                deadline_ns=rng.integers(1, 1 << 40, total).astype(np.uint64),
                lost=(rng.random(total) < 0.01).astype(np.uint8),
                kv_capacity=np.full(S, cap_kv, np.int32) + rng.integers(0, max(1, cap_kv // 2), S).astype(np.int32),
                batch_cap=None if cap_batch is None else np.full(S, cap_batch, np.int32))


@pytest.mark.parametrize("unsorted", [False, True])
@pytest.mark.parametrize("S,H,N,R,Q,cap_kv,cap_batch", [
    (3, 200, 16, 8, 63, 400, None), (3, 64, 16, 0, 128, 300, None), (2, 257, 64, 20, 129, 1 << 20, None),
    (2, 1000, 16, 40, 1500, 900, None), (2, 1000, 24, 40, 1500, 700, None), (3, 300, 1, 10, 1100, 9000, None),
    (2, 700, 8, 300, 1200, 200, None), (2, 500, 100, 5, 1300, 150, None), (2, 400, 16, 12, 300, 5000, 20),
])
def test_queue_paths(S, H, N, R, Q, cap_kv, cap_batch, unsorted):
    inp = _boards(H + Q, S, H, N, R, Q, cap_kv, cap_batch, unsorted)
    assert_projection_equal(gpu_project(inp), oracle.project(inp))


@pytest.mark.parametrize("S,H,N,R,Q,cap_kv,cap_batch", [
    (2, 600, 16, 12, 300, 5000, 20), (256, 512, 16, 30, 90, 1400, 32), (257, 513, 64, 30, 90, 400, 32),
    (3, 1100, 24, 40, 260, 1 << 20, 40), (2, 511, 100, 9, 130, 300, 9), (2, 800, 1, 16, 140, 12000, 24),
])
def test_batch_cap_paths(S, H, N, R, Q, cap_kv, cap_batch):
    """Behind a batch cap, on each side of the rule for one or four wavefronts a
    board, the batch full, the capacity binding, or both."""
    inp = _boards(H + Q, S, H, N, R, Q, cap_kv, cap_batch, S % 2 == 1)
    assert_projection_equal(gpu_project(inp), oracle.project(inp))


def test_many_long_queues():
    inp = _boards(5, 2100, 90, 16, 4, 1030, 3000, None, False)
    assert_projection_equal(gpu_project(inp), oracle.project(inp))
