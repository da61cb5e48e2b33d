"""Chunk-first blocks at their edges: rows around the 16-row block, token
counts around the 16-token wavefront slices and 64-token blocks, one chunk and
several per chain, with and without private chunks (the launch of chunk-first
work alone), both data types, against the oracle."""
import numpy as np
import pytest

from parity_util import Pair, assert_close

pytestmark = pytest.mark.gpu


def _check(c, H, d, dt, rows, prompt, own, seg, scale=0.0, spike=False):
    rng = np.random.default_rng(rows * 1000 + prompt)
    p = Pair(c, H, d, dt, -(-prompt // c) + rows * (-(-max(own, 1) // c) + 2) + 4)
    kp = rng.standard_normal((2, prompt, H, d)).astype(dt)
    if spike:  # scores far apart: the reference maximum moves, and late
        kp[0] *= np.linspace(0.1, 6, prompt)[:, None, None].astype(dt)
    for sid in range(rows):
        kv = np.concatenate([kp, rng.standard_normal((2, own, H, d)).astype(dt)], axis=1)
        p.insert(sid, list(range(prompt)) + [10_000 * (sid + 1) + i for i in range(own)], kv[0], kv[1])
    if seg:
        p.cache.set_tuning(seg_chunks=seg)
    q = {sid: rng.standard_normal((H, d)).astype(dt) for sid in range(rows)}
    for rep in range(2):
        o, qs, row_seq = p.attention(q, scale=scale)
        assert_close(o, p.reference(row_seq, qs, scale), dt,
                     f"c={c} d={d} {np.dtype(dt).name} rows={rows} prompt={prompt} own={own} seg={seg}")


@pytest.mark.parametrize("dt", [np.float32, np.float16])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("c,rows,prompt,own,seg", [
    (64, 2, 1, 0, 0),          # one token
    (64, 16, 64, 0, 0),        # one full block
    (64, 17, 64 + 15, 1, 0),   # a second row block of one row; a slice short by one
    (64, 15, 3 * 64 + 17, 3, 1),
    (64, 33, 7 * 64, 0, 3),    # three row blocks; uneven chains
    (64, 32, 5 * 64 + 33, 70, 64),
    (100, 5, 350, 0, 2),       # chunks of two blocks, the second short
    (128, 19, 300, 129, 0),
])
def test_edges(dt, d, c, rows, prompt, own, seg):
    print(f"[case] chunk-first {np.dtype(dt).name} d={d} c={c} rows={rows} prompt={prompt} own={own}", flush=True)
    _check(c, 2, d, dt, rows, prompt, own, seg)


@pytest.mark.parametrize("dt", [np.float32, np.float16])
def test_moving_reference_maximum(dt):
    print(f"[case] chunk-first spikes {np.dtype(dt).name}", flush=True)
    _check(64, 2, 128, dt, 18, 400, 10, 0, scale=0.3, spike=True)


@pytest.mark.parametrize("dt", [np.float32, np.float16])
@pytest.mark.parametrize("c,d,rows,prompt,own", [
    (1, 64, 3, 20, 150),      # 64 chunks a step, past one group of 64
    (5, 128, 2, 33, 77),      # 12 chunks a step, four idle token places
    (7, 64, 4, 0, 460),       # nothing shared, past one group of 64
    (8, 128, 17, 100, 9),     # the most inline slots a first step can need
    (10, 128, 5, 45, 200),
    (16, 128, 33, 16 * 9, 16 * 5 + 1),
    (16, 64, 2, 1, 1),
    (17, 128, 6, 17 * 5 + 3, 40),   # two chunks a chunk-first step, three private ones
    (31, 64, 18, 200, 100),
    (32, 128, 16, 32 * 70, 32 * 3),  # more than one segment of 64
    (33, 128, 3, 100, 70),    # the smallest chunk the plain path takes
    (48, 64, 3, 150, 100),
])
def test_small_chunks(dt, c, d, rows, prompt, own):
    """Chunks of at most 32 tokens share a step; ragged private lists, short
    chunks mid-path (a prefix that ends inside a chunk), last chunks that grow,
    and rows past a chunk's length that hold NaN."""
    print(f"[case] small chunks {np.dtype(dt).name} c={c} d={d} rows={rows} prompt={prompt} own={own}", flush=True)
    H = 2
    rng = np.random.default_rng(c * 100 + rows)
    p = Pair(c, H, d, dt, -(-prompt // c) + rows * (-(-(own + 12) // c) + 3) + 8)
    for pool in (p.cache.k_pool, p.cache.v_pool):
        pool.fill_(float("nan"))
    kp = rng.standard_normal((2, prompt, H, d)).astype(dt)
    for sid in range(rows):
        n = max(1, own - (sid * own) // (2 * rows))
        kv = np.concatenate([kp, rng.standard_normal((2, n, H, d)).astype(dt)], axis=1)
        p.insert(sid, list(range(prompt)) + [10_000 * (sid + 1) + i for i in range(n)], kv[0], kv[1])
    ids = list(range(rows))
    for step in range(4):
        q = {sid: rng.standard_normal((H, d)).astype(dt) for sid in ids}
        o, qs, row_seq = p.attention(q)
        assert_close(o, p.reference(row_seq, qs, 0.0), dt, f"c={c} step {step}")
        for _ in range(3):
            kv = rng.standard_normal((2, rows, H, d)).astype(dt)
            p.append(ids, [7] * rows, kv[0], kv[1])
        if step == 1:
            p.cache.set_tuning(schedule=0)
        if step == 2:
            p.cache.set_tuning(schedule=2, split_chunks=2)
