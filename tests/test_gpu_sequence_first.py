"""Calls without a shared chunk (sequence-first work alone) around the number
of blocks up to which fp32 with d = 128 takes the sequence-first kernel itself
(2,048 on 256 compute units), rows whole and cut, against the oracle."""
import numpy as np
import pytest
import torch

from parity_util import Pair, assert_close, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt,d,c,rows,H,own", [
    (np.float32, 128, 64, 1, 3, 1),
    (np.float32, 128, 64, 64, 32, 70),    # 2,048 blocks
    (np.float32, 128, 64, 65, 32, 70),    # 2,080
    (np.float32, 128, 100, 5, 4, 900),    # cut rows: pieces counted and folded in the launch
    (np.float32, 128, 33, 7, 2, 300),
    (np.float32, 128, 32, 8, 4, 200),     # small chunks stay with the fused kernel
    (np.float32, 64, 64, 6, 4, 500),
    (np.float16, 128, 64, 6, 4, 500),
])
def test_private_only(dt, d, c, rows, H, own):
    print(f"[case] private only {np.dtype(dt).name} d={d} c={c} rows={rows} H={H} own={own}", flush=True)
    rng = np.random.default_rng(rows * own)
    p = Pair(c, H, d, dt, rows * (-(-own // c) + 2))
    for sid in range(rows):
        n = max(1, own - 3 * sid)
        kv = rng.standard_normal((2, n, H, d)).astype(dt)
        p.insert(sid, 10_000 * (sid + 1) + np.arange(n), kv[0], kv[1])
    q = {sid: rng.standard_normal((H, d)).astype(dt) for sid in range(rows)}
    for sched in (2, 1, 0):
        p.cache.set_tuning(schedule=sched)
        for _ in range(2):  # the counters are left at zero
            o, qs, row_seq = p.attention(q)
            ref = p.reference(row_seq, qs, 0.0)
            assert_close(o, ref, dt, f"schedule {sched}")
    p.cache.set_tuning(schedule=2)
    ids = np.random.default_rng(1).permutation(rows)
    o = p.cache.attention(to_dev(np.stack([q[int(s)] for s in ids])), seq_ids=ids).cpu().numpy()
    at = {int(s): i for i, s in enumerate(ids)}
    assert_close(o[[at[int(s)] for s in row_seq]], ref, dt, "caller order")
