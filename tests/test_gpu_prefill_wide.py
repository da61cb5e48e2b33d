"""Prefill with 32-query wavefronts (joins whose query tiles give every compute
unit a block): both tile sizes, ragged tiles, chunks of 1 to 130 tokens (paths
in the argument table, past one 64-chunk window, and on the device), short
chunks mid-path, both head sizes and layouts, against the oracle. The pool is
poisoned with NaN first, so a row read past a chunk's length shows."""
import numpy as np
import pytest
import torch

from oracle import prefill_attention
from parity_util import Pair, assert_close, to_dev
from workloads import prefix_keyed_kv

pytestmark = pytest.mark.gpu


# heads x ceil(n_q / 128) >= 256 blocks (compute units): 128-query tiles, at
# d = 64 only in three rounds or, from 448 blocks on, with 2/7 of the path cached,
# and not in chunks that part fill the units; else, if heads x ceil(n_q / 64) >
# 256 (d = 64: where the 128-query tiles were in question), 64-query tiles; over
# chunks of at most 32 tokens a model decides
@pytest.mark.parametrize("c,d,H,prefix,n_q,layout", [
    (64, 128, 128, 100, 129, "interleaved"),   # 128-query tiles, the last of one query
    (64, 64, 256, 0, 77, "split"),             # nothing cached: 64-query tiles
    (64, 64, 256, 0, 300, "interleaved"),      # 768 128-query tiles
    (64, 64, 256, 120, 200, "split"),          # 512, 3/8 cached
    (16, 64, 256, 100, 200, "interleaved"),    # four chunks a unit, d = 64
    (32, 64, 256, 100, 200, "split"),          # two
    (48, 64, 256, 120, 200, "split"),          # units part masked: 64-query tiles
    (48, 64, 256, 30, 70, "interleaved"),      # the same, 256: 16-query blocks
    (16, 128, 128, 37, 200, "interleaved"),    # a short chunk mid-path
    (130, 64, 128, 300, 140, "split"),         # five 32-row units a chunk, the last of two rows
    (130, 128, 128, 300, 140, "split"),        # three 64-row units a chunk, the last of two rows
    (3, 128, 128, 50, 250, "interleaved"),     # 100 chunks: past one window
    (1, 64, 256, 200, 100, "split"),           # 300 chunks: device table
    (64, 128, 130, 100, 65, "split"),          # 64-query tiles, two key groups
    (64, 128, 128, 100, 65, "split"),          # 256 64-query tiles: 16-query blocks
    (64, 128, 32, 2480, 512, "interleaved"),   # the same over a longer path
    (64, 128, 32, 2488, 512, "split"),
    (64, 128, 32, 2487, 513, "split"),         # 288: 64-query tiles
    (16, 64, 128, 1, 128, "interleaved"),      # 64-query tiles, 32-row units
    (100, 128, 256, 5, 20, "interleaved"),     # 128-query tile, mostly past n_q
    (7, 128, 130, 400, 70, "split"),           # 64-query tiles past one window
    (2, 64, 128, 460, 90, "interleaved"),      # 275 chunks, 64-query tiles
    (200, 128, 130, 30, 100, "split"),         # 64-query tiles, seven 32-row units a chunk
    (32, 128, 128, 70, 150, "interleaved"),    # two chunks a unit, one short inside
    (32, 64, 128, 70, 100, "split"),           # one 32-token chunk a 32-row unit
    (16, 128, 128, 1100, 130, "split"),        # four chunks a unit, past one window
    (16, 64, 256, 21, 90, "split"),
    (16, 128, 128, 5, 100, "interleaved"),     # two chunks a unit, the first short
    (16, 128, 256, 0, 3, "split"),             # one chunk in all
    (64, 128, 32, 1030, 130, "interleaved"),   # 16-query blocks: two parts, one round
    (64, 128, 32, 4000, 300, "split"),         # three parts, two rounds
    (16, 128, 32, 500, 257, "interleaved"),    # small chunks: 64-query tiles from half the chip on
    (64, 64, 128, 30, 128, "split"),           # d = 64, 256 64-query tiles: 16-query blocks
])
def test_wide_tiles(c, d, H, prefix, n_q, layout):
    print(f"[case] prefill wide c={c} d={d} H={H} prefix={prefix} n_q={n_q} {layout}", flush=True)
    rng = np.random.default_rng(c * 1000 + n_q)
    p = Pair(c, H, d, np.float16, 2 * (prefix + n_q) // c + 80, layout=layout)
    for pool in (p.cache.k_pool, p.cache.v_pool):
        pool.fill_(float("nan"))
    pre = rng.integers(0, 50, prefix).astype(np.int32)
    for sid, tail in ((0, np.full(9, 60)), (1, rng.integers(70, 90, n_q))):
        toks = np.concatenate([pre, tail]).astype(np.int32)
        k, v = prefix_keyed_kv(5, toks, 0, H, d, np.float16)
        p.insert(sid, toks, k, v)
    q = rng.standard_normal((n_q, H, d)).astype(np.float16)
    rows = sorted({0, n_q - 1, n_q // 2, min(63, n_q - 1), min(64, n_q - 1), min(31, n_q - 1)}
                  | {int(x) for x in rng.integers(0, n_q, 6)})
    for scale in (0.0, 0.4):
        o = p.cache.prefill(1, to_dev(q), scale=scale).cpu().numpy()
        ref = prefill_attention(p.tree, 1, q, scale or 1.0 / np.sqrt(d), queries=rows)
        assert_close(o[rows], ref, np.float16, f"wide c={c} d={d} H={H} n_q={n_q} scale={scale}")
        assert np.isfinite(o).all()


def test_moving_reference_maximum():
    """Scores that grow along the path by far more than the slack of the
    softmax reference: every unit moves it."""
    print("[case] prefill wide spikes", flush=True)
    c, d, H, n_q = 64, 128, 128, 150
    rng = np.random.default_rng(3)
    p = Pair(c, H, d, np.float16, 40)
    n = 500
    toks = np.arange(n, dtype=np.int32)
    k = (rng.standard_normal((n, H, d)) * np.linspace(0.05, 2, n)[:, None, None]).astype(np.float16)
    v = rng.standard_normal((n, H, d)).astype(np.float16)
    p.insert(0, toks, k, v)
    q = (3 * rng.standard_normal((n_q, H, d))).astype(np.float16)
    o = p.cache.prefill(0, to_dev(q), scale=0.2).cpu().numpy()
    rows = [0, 1, 31, 32, 100, 127, 128, 149]
    ref = prefill_attention(p.tree, 0, q, 0.2, queries=rows)
    # a peaked softmax passes single V rows through: fp16 rounding of values up
    # to ~4.5 (half an ulp 2e-3) on top of the probabilities' own
    err = np.abs(o[rows].astype(np.float64) - ref)
    print(f"[parity] spikes max_abs={err.max():.3e}", flush=True)
    assert (err <= 2e-3 + 2.0 ** -10 * np.abs(ref)).all()


@pytest.mark.parametrize("d", [64, 128])
# 128-query tiles (d = 64: of 768 heads), 64-query tiles or 16-query blocks, 128-query tiles
@pytest.mark.parametrize("H,c", [(256, 16), (768, 16), (128, 16), (256, 32)])
@pytest.mark.parametrize("prefix,n_q", [(5, 3), (5, 8), (1, 10), (5, 16), (13, 16), (13, 30), (1, 40), (31, 9)])
def test_units_that_end_past_the_path(c, H, d, prefix, n_q):
    """A short first chunk, one or two more, and places of the unit past the
    path's end: those hold no token for any query, the earliest positions
    included. Every query is compared."""
    print(f"[case] prefill wide short path c={c} H={H} d={d} prefix={prefix} n_q={n_q}", flush=True)
    p = Pair(c, H, d, np.float16, 16)
    pre = np.arange(prefix, dtype=np.int32)
    for sid, tail in ((0, np.full(2, 90)), (1, 100 + np.arange(n_q))):
        toks = np.concatenate([pre, tail]).astype(np.int32)
        k, v = prefix_keyed_kv(7, toks, 0, H, d, np.float16)
        p.insert(sid, toks, k, v)
    for n in (n_q, prefix + n_q):  # the new tokens; the whole path from position 0
        q = np.random.default_rng(n).standard_normal((n, H, d)).astype(np.float16)
        o = p.cache.prefill(1, to_dev(q)).cpu().numpy()
        assert_close(o, prefill_attention(p.tree, 1, q, 1.0 / np.sqrt(d)), np.float16, f"n={n}")


@pytest.mark.parametrize("c,d,H,n_q", [
    (64, 64, 192, 512),    # 128-query tiles
    (64, 128, 64, 512),
    (16, 128, 64, 512),    # the same, four chunks a unit
    (16, 64, 2, 70),       # 64-query tiles, two chunks a unit
    (64, 128, 65, 250),    # 64-query tiles
    (64, 64, 2, 70),       # 16-query blocks
])
def test_long_flat_tail_below_a_peak(c, d, H, n_q):
    """One token far above a long tail whose probabilities, about 2^-16 of the
    peak's, are subnormal in fp16: the row's sum and the product with V have to
    treat them alike. Dropped from either side they would move o by ~0.04."""
    print(f"[case] prefill wide flat tail c={c} d={d} H={H} n_q={n_q}", flush=True)
    n = 3000 if H < 100 else 1500
    rng = np.random.default_rng(d + n_q)
    p = Pair(c, H, d, np.float16, -(-n // c) + 4)
    k = (rng.standard_normal((n, H, d)) * 0.02).astype(np.float16)
    k[:, :, 0] = 0
    k[3, :, 0] = 4
    v = (1 + 0.1 * rng.standard_normal((n, H, d))).astype(np.float16)
    v[3] = 0
    toks = np.arange(n, dtype=np.int32)
    p.insert(0, toks, k, v)
    q = (rng.standard_normal((n_q, H, d)) * 0.5).astype(np.float16)
    q[:, :, 0] = 4
    scale = float(np.log(2.0))  # scores in powers of two: 16 at the peak, about 0 elsewhere
    o = p.cache.prefill(0, to_dev(q), scale=scale).cpu().numpy()
    rows = [0, 1, 31, 32, 63, n_q - 1]
    ref = prefill_attention(p.tree, 0, q, scale, queries=rows)
    err = np.abs(o[rows].astype(np.float64) - ref).max()
    print(f"[parity] flat tail max_abs={err:.3e} o={np.abs(ref).mean():.3f}", flush=True)
    # each probability is rounded to a multiple of 2^-24, half of one at most:
    # n of them in the sum and, times |V| < 1.5, in the product; o itself to fp16
    assert 0.015 < np.abs(ref).mean() < 0.2
    assert err <= 2.5 * n * 2.0 ** -25 + 2.0 ** -11 * np.abs(ref).max()
