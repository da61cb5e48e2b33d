"""Automatic split of long private lists (the default schedule): the plan,
seen through the workspace size, decode growth on cut rows, and the results of
cut rows against the oracle."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from parity_util import Pair, assert_close
from paper_2402_15220_amd import binding as B


def _align(x, a=256):
    return (x + a - 1) // a * a


def _ws(parts, H, d):
    return _align(parts * H * d * 4) + _align(parts * H * 2 * 4)


def _table_cache(c, H, d, slots=1 << 16, check=False):
    if check:
        os.environ["CA_CHECK_PATCH"] = "1"
    try:
        return B.ca_create(c, H, d, B.CA_FP16, slots)
    finally:
        os.environ.pop("CA_CHECK_PATCH", None)


# 256 compute units: a piece is ceil(total steps * H / 256) steps, at least 2; a
# row is cut when that takes at least 8 steps off it (d = 64, fp16, nothing
# shared) and its chain takes longer than all bytes
@pytest.mark.parametrize("c,H,lens,parts", [
    (64, 32, [32765], 8),            # 512 steps: pieces of 64
    (64, 32, [5 * 64], 0),           # 5 steps, pieces of 2: 3 saved, whole
    (64, 32, [6 * 64], 0),           # 6 steps: 4 saved, whole (5.3 us, 6.6 in 3 pieces)
    (64, 32, [9 * 64], 0),           # 7 saved
    (64, 32, [10 * 64], 5),          # 8 saved
    (64, 64, [64 * 30] * 3, 6),      # 192 blocks: pieces of 23
    (64, 84, [64 * 30] * 3, 0),      # 252: the chip's read rate is the limit
    (48, 4, [250], 0),               # six chunks are six steps
    (64, 1, [64 * 512], 64),         # 256 pieces of 2 would be over the 64 a row may have
    (64, 256, [64 * 4096], 0),       # every compute unit has a whole head
    (16, 32, [32 * 64], 8),          # 128 chunks of 16 are 32 steps: pieces of 4
    (128, 32, [32 * 64], 8),         # 16 chunks of 128 likewise
    (64, 32, [64 * 300] + [64] * 8, 8),   # 308 steps: pieces of 39, the long row only
    (300, 8, [300 * 2], 0),          # two chunks of 5 steps: 5 saved
    (300, 8, [300 * 3], 3),          # more pieces wanted than chunks
    (256, 8, [256 * 2 + 5], 0),      # 9 steps, not 12: three pieces save 5
])
def test_plan(c, H, lens, parts):
    h = _table_cache(c, H, 64)
    tok = 0
    for sid, n in enumerate(lens):
        B.ca_insert(h, sid, np.arange(tok, tok + n))
        tok += n
    assert B.ca_workspace_size(h) == _ws(parts, H, 64)
    B.ca_set_tuning(h, split_chunks=0)       # an explicit 0 disables it
    assert B.ca_workspace_size(h) == 0
    B.ca_set_tuning(h, split_chunks=-1)      # kept
    assert B.ca_workspace_size(h) == 0
    B.ca_set_tuning(h, split_chunks=-2)      # automatic again
    assert B.ca_workspace_size(h) == _ws(parts, H, 64)
    with pytest.raises(B.ChunkAttnError):
        B.ca_set_tuning(h, split_chunks=-3)
    B.ca_destroy(h)
    h = _table_cache(c, H, 64)
    B.ca_insert(h, 0, np.arange(lens[0]))
    B.ca_set_tuning(h, schedule=0)           # other schedules keep rows whole
    assert B.ca_workspace_size(h) == 0
    B.ca_destroy(h)


# fp32, d = 128: pieces rounded down to a block per compute unit, rows cut for
# four steps, nothing cut where all bytes take as long as the longest row
@pytest.mark.parametrize("c,H,rows,own,prompt,parts", [
    (128, 1, 86, 2570, 0, 172),      # 41 steps, pieces of 14: two, not three (258 blocks)
    (64, 8, 19, 3104, 0, 0),         # 152 blocks read at the chip's rate
    (64, 32, 1, 6 * 64, 0, 3),       # 4 steps saved
    (64, 32, 1, 5 * 64, 0, 0),
    (64, 8, 4, 12 * 64, 1024, 16 * 4 + 4 * 3),   # 16 segments on the path: pieces of four steps
    (64, 8, 4, 12 * 64, 128, 2 * 4 + 4 * 6),     # 2 segments: of two
])
def test_plan_fp32(c, H, rows, own, prompt, parts):
    h = B.ca_create(c, H, 128, B.CA_FP32, 1 << 13)
    for sid in range(rows):
        B.ca_insert(h, sid, list(range(prompt)) + list(range(100_000 * (sid + 1), 100_000 * (sid + 1) + own)))
    B.ca_set_tuning(h, seg_chunks=1)
    assert B.ca_workspace_size(h) == _ws(parts, H, 128)
    B.ca_destroy(h)


@pytest.mark.parametrize("H,rows", [(1, 1), (4, 3), (64, 5)])
def test_growth_patches_cut_rows(H, rows):
    """Growth extends a cut row's last piece in place, each patch equal to a
    rebuild; when the piece has doubled, the row is planned again."""
    h = _table_cache(2, H, 64, check=True)
    for sid in range(rows):
        B.ca_insert(h, sid, np.arange(1000 * sid, 1000 * sid + 900))
    B.ca_seq_order(h)
    sizes = {B.ca_workspace_size(h)}
    for step in range(1200):
        B.ca_append_batch(h, np.arange(rows), np.full(rows, 7))
        B.ca_seq_order(h)
        B.ca_stats(h)
        sizes.add(B.ca_workspace_size(h))
    st = B.ca_stats(h)
    assert st["patches"] > 550               # one per new chunk of every row, few rebuilds
    assert len(sizes) <= 4
    B.ca_destroy(h)


def test_patch_check_finds_planted_mistakes(tmp_path):
    """The comparison of a patched list with a rebuilt one, on lists with cut
    rows: wrong, missing, doubled or misnumbered pieces and partials."""
    if shutil.which("g++") is None:
        pytest.skip("no g++ in this image")
    here = os.path.dirname(os.path.abspath(__file__))
    csrc = os.path.join(os.path.dirname(here), "paper_2402_15220_amd", "csrc")
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-std=c++17", "-O1", f"-I{csrc}", os.path.join(here, "work_lists_check.cpp"),
                    os.path.join(csrc, "tables.cpp"), os.path.join(csrc, "tree.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "", r.stdout + r.stderr


@pytest.mark.parametrize("H,parts", [(128, 248), (64, 249)])
def test_static_scratch_never_outgrown_by_the_split(H, parts):
    """31 rows over 7 segments: 248 partials. With 128 heads they fill the
    static scratch (16,515,072 bytes) to within one, so the long row stays
    whole; with 64 heads there is room and it is cut in two."""
    d = 128
    h = _table_cache(1, H, d)
    for sid in range(30):
        B.ca_insert(h, sid, list(range(64 * 7)) + [10_000 + sid])
    B.ca_insert(h, 30, list(range(64 * 7)) + [20_000 + i for i in range(3000 if H == 128 else 1500)])
    B.ca_set_tuning(h, seg_chunks=64)
    assert B.ca_workspace_size(h) == _ws(parts, H, d)
    B.ca_destroy(h)


# shared runs of a tree too small to fill the chip: at most about 16 segments a
# run, counted in steps of as many small chunks as a block works on at once
@pytest.mark.parametrize("c,H,rows,prompt,seg", [
    (64, 1, 8, 64 * 16, 1),      # 16 chunks: a quota of one, 16 segments
    (64, 1, 8, 64 * 17, 2),
    (64, 1, 8, 64 * 64, 4),
    (64, 1, 8, 64 * 1000, 16),   # no longer than that for its own sake
    (16, 1, 8, 16 * 64, 4),      # 16 steps of four chunks
    (16, 1, 8, 16 * 65, 8),
    (32, 1, 8, 32 * 64, 4),      # 32 steps of two
])
def test_smallest_segments(c, H, rows, prompt, seg):
    h = _table_cache(c, H, 64)
    for sid in range(rows):
        B.ca_insert(h, sid, list(range(prompt)) + [100_000 + sid])
    B.ca_workspace_size(h)
    assert B.ca_stats(h)["seg_chunks"] == seg
    B.ca_destroy(h)


# longer segments of a small tree pay while their length squared, times a
# chunk's cost in 512-byte steps of 64 tokens, is below 0.8 of the run, and only
# where the launch itself finishes the rows (schedules 2 and 3)
@pytest.mark.parametrize("c,dt,chunks,schedule,seg", [
    (200, B.CA_FP32, 32, 2, 1),      # a chunk costs 8: two would be 32, over 25.6
    (200, B.CA_FP32, 80, 2, 2),
    (200, B.CA_FP16, 80, 2, 4),
    (256, B.CA_FP16, 63, 2, 2),
    (64, B.CA_FP32, 100, 2, 4),
    (64, B.CA_FP32, 250, 3, 8),
    (64, B.CA_FP16, 64, 3, 4),
    (64, B.CA_FP16, 64, 0, 1),
    (64, B.CA_FP16, 64, 1, 1),
    (16, B.CA_FP16, 64, 0, 4),       # one step of four small chunks
])
def test_smallest_segments_weigh_the_chain(c, dt, chunks, schedule, seg):
    h = B.ca_create(c, 1, 128, dt, 1 << 12)
    B.ca_set_tuning(h, schedule=schedule)
    for sid in range(3):
        B.ca_insert(h, sid, list(range(c * chunks)) + [100_000 + sid])
    B.ca_workspace_size(h)
    assert B.ca_stats(h)["seg_chunks"] == seg
    B.ca_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("c,H,d,dt,prompt,lens", [
    (64, 2, 128, np.float16, 0, [64 * 6 + 1]),
    (64, 1, 64, np.float16, 0, [64 * 130 + 7]),       # more than 64 pieces wanted
    (16, 3, 128, np.float16, 40, [1500, 90, 700]),    # a shared prompt: chunk-first partials too
    (100, 2, 64, np.float32, 0, [2001, 640]),
    (5, 1, 128, np.float32, 12, [900, 1]),
    (64, 4, 128, np.float16, 4200, [3000, 2000]),     # more than 64 partials a row (seg 1 below)
])
def test_cut_rows_against_the_oracle(c, H, d, dt, prompt, lens):
    print(f"[case] split c={c} H={H} d={d} {np.dtype(dt).name} prompt={prompt} lens={lens}", flush=True)
    rng = np.random.default_rng(c * H + d)
    steps = 40
    slots = sum(-(-(n + steps) // c) + 2 for n in lens + [prompt])
    p = Pair(c, H, d, dt, slots)
    kp = rng.standard_normal((2, prompt, H, d)).astype(dt)
    for sid, n in enumerate(lens):
        own = rng.standard_normal((2, n, H, d)).astype(dt)
        kv = np.concatenate([kp, own], axis=1)
        p.insert(sid, list(range(prompt)) + [100_000 * (sid + 1) + i for i in range(n)], kv[0], kv[1])
    if prompt > 4000:
        p.cache.set_tuning(seg_chunks=1)
    ids = list(range(len(lens)))
    for step in range(3):
        q = {sid: rng.standard_normal((H, d)).astype(dt) for sid in ids}
        o, qs, row_seq = p.attention(q)
        assert_close(o, p.reference(row_seq, qs, 0.0), dt, f"step {step}")
        out = torch.empty(qs.shape, dtype=torch.from_numpy(qs).dtype, device="cuda")
        o2 = p.cache.attention_noalloc(torch.from_numpy(qs).cuda(), out)
        torch.cuda.synchronize()
        assert_close(o2.cpu().numpy(), o, dt, "noalloc")
        for _ in range(steps // 2 if step < 2 else 0):  # growth patches the last pieces
            kv = rng.standard_normal((2, len(ids), H, d)).astype(dt)
            p.append(ids, [7] * len(ids), kv[0], kv[1])


@pytest.mark.gpu
@pytest.mark.parametrize("prompt,rows", [(0, 1), (200, 3)])
def test_workspace_without_the_split(prompt, rows):
    """A workspace that holds the partials of whole rows (none at all without
    shared chunks) is accepted however far the rows grow; a smaller one is
    refused and changes nothing."""
    print(f"[case] workspace without the split prompt={prompt} rows={rows}", flush=True)
    c, H, d, own = 64, 2, 128, 600
    rng = np.random.default_rng(prompt + rows)
    p = Pair(c, H, d, np.float16, 80)
    whole = _table_cache(c, H, d)
    B.ca_set_tuning(whole, split_chunks=0)
    kp = rng.standard_normal((2, prompt, H, d)).astype(np.float16)
    for sid in range(rows):
        kv = np.concatenate([kp, rng.standard_normal((2, own, H, d)).astype(np.float16)], axis=1)
        toks = list(range(prompt)) + [10_000 * (sid + 1) + i for i in range(own)]
        p.insert(sid, toks, kv[0], kv[1])
        B.ca_insert(whole, sid, toks)
    need = B.ca_workspace_size(whole)
    B.ca_destroy(whole)
    assert (need > 0) == (prompt > 0)
    ws = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda")
    s = p.cache.stream()

    def attend(size):
        row_seq = p.cache.seq_order()
        q = rng.standard_normal((rows, H, d)).astype(np.float16)
        qd, o = torch.from_numpy(q).cuda(), torch.empty((rows, H, d), dtype=torch.float16, device="cuda")
        B.ca_attention(p.cache.h, qd.data_ptr(), o.data_ptr(), 0.0, ws.data_ptr() if size else 0, size, s)
        torch.cuda.synchronize()
        assert_close(o.cpu().numpy(), p.reference(row_seq, q, 0.0), np.float16, f"ws={size}")

    cut = B.ca_workspace_size(p.cache.h)
    assert cut > need
    if need:
        with pytest.raises(B.ChunkAttnError) as ei:
            attend(need - 1)
        assert ei.value.status == B.CA_ERR_WORKSPACE
        assert B.ca_workspace_size(p.cache.h) == cut
    attend(need)
    ids = list(range(rows))
    for step in range(3 * c):
        kv = rng.standard_normal((2, rows, H, d)).astype(np.float16)
        p.append(ids, [7] * rows, kv[0], kv[1])
        if step % 50 == 0 or step == 3 * c - 1:
            attend(need)
    p.remove(0)  # a structural change plans the split again
    if rows > 1:
        rows -= 1
        assert B.ca_workspace_size(p.cache.h) > 0
        ids = list(p.cache.seq_order())
        attend(need)
