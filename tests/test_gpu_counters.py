"""Arrival counters of the partial-writing schedules: a line each up to 512
(row, head) pairs, 16 rows of a head a line above, packed where that would not
fit 65,536 entries; every layout against the oracle, twice (the kernels reset
the counters they used)."""
import numpy as np
import pytest
import torch

from parity_util import Pair, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,H", [(8, 64), (9, 57), (37, 65), (513, 64), (512, 64)])
def test_counter_layouts(rows, H):
    print(f"[case] counters rows={rows} H={H}", flush=True)
    d, c = 64, 8
    rng = np.random.default_rng(rows * H)
    p = Pair(c, H, d, np.float16, 3 * rows + 8)
    prompt = list(range(20))
    kp = rng.standard_normal((2, len(prompt), H, d)).astype(np.float16)
    for sid in range(rows):
        own = rng.standard_normal((2, 3, H, d)).astype(np.float16)
        kv = np.concatenate([kp, own], axis=1)
        p.insert(sid, prompt + [1000 + sid, 1, 2], kv[0], kv[1])
    q = {sid: rng.standard_normal((H, d)).astype(np.float16) for sid in range(rows)}
    some = sorted(rng.choice(rows, min(rows, 12), replace=False))
    for rep in range(2):
        o, qs, row_seq = p.attention(q)
        ref = p.reference(row_seq, qs, 0.0, rows=some)
        assert_close(o[some], ref, np.float16, f"counters rows={rows} H={H} call {rep}")
        if rep == 0:
            # the same call from the static scratch
            out = p.cache.attention_noalloc(torch.from_numpy(qs).cuda(), torch.empty(qs.shape, dtype=torch.float16, device="cuda")) \
                if rows * H <= 65536 and rows * H * d * 4 * 4 < 15 << 20 else None
            if out is not None:
                torch.cuda.synchronize()
                assert_close(out.cpu().numpy()[some], ref, np.float16, "noalloc")
