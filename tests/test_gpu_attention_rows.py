"""Attention of new turns and recomputed contexts of small batches, against the oracle: rows, keys and pages
at and beside their edges, items that leave some of the kernel's wavefronts without rows; and a new turn's
independence from what it runs with."""
import numpy as np
import pytest

from gpu_util import decode_pages, kv_tolerance_ok, stack_kv
from oracle import transformer as T
from workloads import SHAPES, WeightSource

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape_name, n_ctx, n_new", [
    ("mini-bf16", [1, 15, 16, 31, 33, 130], [1, 16, 17, 2, 31, 128]),
    ("mini-bf16", [3, 129, 63] + [20] * 15, [33, 1, 16] + [2] * 15),                 # many items
    ("mini64-gqa2-bf16", [47, 64, 1, 100], [1, 15, 33, 65]),
    ("mini128-gqa3-bf16", [32, 17, 96], [16, 5, 32]),
    ("mini64-bf16", [16, 70], [48, 1]),
    ("mini-bf16", [32, 33, 64, 65, 96, 97, 128], [1] * 7),                           # contexts: 1 to 4 wavefronts with rows
    ("mini64-gqa2-bf16", [129, 161, 193, 225], [1] * 4),
    ("mini128-gqa3-bf16", [97, 192], [1, 1])])
def test_new_turn_rows_match_the_oracle(shape_name, n_ctx, n_new):
    """2e-2 on the logits and on the cells, the stated bound of the bf16 models.  The pool starts as NaN
    patterns, so a slot past a request's last key must not reach any result."""
    from paper_2604_25080_amd.runtime import Session
    shape = SHAPES[shape_name]
    ws = WeightSource(shape, 21, cache=True)
    rng = np.random.default_rng(len(n_ctx) + sum(n_new))
    ctx, new = ([rng.integers(0, shape.vocab, size=n).astype(np.int32) for n in v] for v in (n_ctx, n_new))
    s = Session(shape, ws, max_batch=len(n_ctx), max_tokens=sum(n_ctx) + sum(n_new), max_positions=512, n_pages=96,
                pool_fill=0xFF)
    for i, (n, m) in enumerate(zip(n_ctx, n_new)):
        s.cache.alloc(1 + i, n + m)
    reqs = [dict(req_id=1 + i, ctx_tokens=ctx[i], new_tokens=new[i]) for i in range(len(n_ctx))]
    logits, _ = s.restore(reqs, [(0, n, shape.n_layers) for n in n_ctx])
    logits = logits.cpu().numpy().astype(np.float64)
    for i, n in enumerate(n_ctx):
        kv_ctx, kv_new, ref = T.full_reference(shape, ws, ctx[i], new[i])
        assert np.abs(logits[i] - ref).max() <= 2e-2, f"request {i}"
        got = decode_pages(shape, s.read_pages(1 + i, n + n_new[i]), n + n_new[i])
        for a, b in zip(got, stack_kv(shape, kv_ctx, kv_new)):
            assert kv_tolerance_ok(shape, a, b)[0], f"request {i}"
    s.close()


def test_a_new_turn_keeps_its_bits_whatever_it_runs_with():
    """Positions below 2048 (from there on key ranges may be split by how full a launch is): the logits of a
    request alone, among 70 others, and among them under the sequential join.  Chunks of 256 rows: their
    borders fall inside new turns."""
    from paper_2604_25080_amd.runtime import Session
    shape = SHAPES["mini-bf16"]
    rng = np.random.default_rng(8)
    n_ctx, n_new = [77, 331, 100, 640, 2016, 2015, 1, 2040] + [16] * 70, [33, 32, 5, 128, 32, 33, 1, 8] + [2] * 70
    ctx, new = ([rng.integers(0, shape.vocab, size=n).astype(np.int32) for n in v] for v in (n_ctx, n_new))
    n_pages = sum(-(-(n + m) // 16) for n, m in zip(n_ctx, n_new))
    s = Session(shape, WeightSource(shape, 22), max_batch=len(n_ctx), max_tokens=sum(n_ctx) + sum(n_new),
                max_positions=2112, n_pages=n_pages, chunk_rows=256, pool_fill=0xFF)
    for i, (n, m) in enumerate(zip(n_ctx, n_new)):
        s.cache.alloc(1 + i, n + m)
    reqs = [dict(req_id=1 + i, ctx_tokens=ctx[i], new_tokens=new[i]) for i in range(len(n_ctx))]
    splits = [(0, n, shape.n_layers) for n in n_ctx]
    alone = [s.restore(reqs[i:i + 1], splits[i:i + 1])[0][0].clone() for i in range(8)]
    for pipelined in (True, False):
        s.ctx.set_pipelined_join(pipelined)
        logits, _ = s.restore(reqs, splits)
        for i, a in enumerate(alone):
            assert bool((a == logits[i]).all()), f"request {i} (pipelined: {pipelined}), {n_new[i]} rows behind {n_ctx[i]}"
    s.close()
