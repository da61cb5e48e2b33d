"""Arrival counters of the partial-writing schedules: a line each up to 512
(row, head) pairs, 16 rows of a head a line above, packed where that would not
fit 65,536 entries; every layout against the oracle, twice (the kernels reset
the counters they used)."""
import numpy as np
import pytest
import torch

from parity_util import Pair, assert_close
from paper_2402_15220_amd import binding as B

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


def _waits(call):
    """True if the call waits for work that is already on the stream."""
    torch.cuda.synchronize()
    end = torch.cuda.Event()
    torch.cuda._sleep(400_000_000)  # over 0.1 s
    end.record()
    call()
    done = end.query()
    torch.cuda.synchronize()
    return done


def test_growing_batches_never_wait():
    """Counters are allocated once: neither a batch that fills up from one row
    nor joins of more tiles make a call wait for the stream."""
    print("[case] counters of a growing batch", flush=True)
    H, d, c = 32, 128, 64
    p = Pair(c, H, d, np.float16, 200, oracle_kv=False)
    n = 24 * c + 1
    gen = torch.Generator(device="cuda").manual_seed(1)
    kv = torch.randn((2, n + 250, H, d), generator=gen, device="cuda", dtype=torch.float16)
    q = torch.randn((250, H, d), generator=gen, device="cuda", dtype=torch.float16)
    out = torch.empty_like(q)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    s = p.cache.stream()
    waited, joins = [], []
    for rows in range(1, 65):
        p.cache.insert(rows, np.append(np.arange(96), 1000 + rows), kv[0, :97], kv[1, :97])
        if rows & (rows - 1) and rows not in (3, 7, 15, 33):
            continue
        p.cache.prepare()
        call = lambda: B.ca_attention(p.cache.h, q.data_ptr(), out.data_ptr(), 0.0, ws.data_ptr(), ws.numel(), s)
        if rows == 1:
            call()
        elif _waits(call):
            waited.append(rows)
    # joins whose key range is split, 32, 64 and 96 tiles; the first also allocates the partials
    for i, new in enumerate((37, 100, 150)):
        toks = np.concatenate([np.arange(96), 5000 * (i + 1) + np.arange(n - 96 + new)])
        p.cache.insert(100 + i, toks, kv[0, :n + new].contiguous(), kv[1, :n + new].contiguous())
        call = lambda: B.ca_prefill_attention(p.cache.h, 100 + i, q.data_ptr(), out.data_ptr(), new, 0.0, s)
        if i == 0:
            call()
        elif _waits(call):
            joins.append(new)
    assert not waited and not joins, f"rows {waited}, joins {joins}"
