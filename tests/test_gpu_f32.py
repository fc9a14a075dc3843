"""The float32 kernels on the matrix cores against their definitions: the GEMM at the edges of its
tiles and K-steps, the paged attention at the edges of its query blocks and pages."""
import numpy as np
import pytest
import torch

from oracle import transformer as T
from workloads import WeightSource
from workloads.shapes import ModelShape

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sess():
    from paper_2604_25080_amd.runtime import Session
    shape = ModelShape("f32-1", 1, 64, 1, 1, 64, 64, 32, 10000.0, 1e-5, "f32")
    s = Session(shape, WeightSource(shape, 5), max_batch=2, max_tokens=64, max_positions=64, n_pages=8)
    yield s
    s.close()


@pytest.mark.parametrize("mnk", [(1, 1, 4), (31, 33, 28), (32, 32, 32), (33, 65, 36), (65, 1000, 688),
                                 (1025, 1021, 132), (2049, 513, 260)])
def test_gemm_f32_matches_float64_matmul(sess, mnk):
    """Bound: a sum of K products in any order is off by at most K * 2^-24 of the sum of their
    magnitudes (SiLU * mul: the same for each factor, and SiLU's slope stays below 1.1)."""
    import paper_2604_25080_amd as cf
    M, N, K = mnk
    g = torch.Generator().manual_seed(M + N + K)
    a, w, w2 = (torch.randn(r, K, generator=g) for r in (M, N, N))
    c0 = torch.randn(M, N, generator=g)
    ref, ref2 = a.double() @ w.double().t(), a.double() @ w2.double().t()
    eps = (K + 4) * 2.0 ** -24
    mag, mag2 = a.double().abs() @ w.double().abs().t(), a.double().abs() @ w2.double().abs().t()
    A, W, W2 = a.cuda(), w.cuda(), w2.cuda()
    silu = ref * torch.sigmoid(ref)
    want = {cf.EPI_STORE_F32: (ref, eps * mag), cf.EPI_ADD_F32: (ref + c0, eps * (mag + (ref + c0).abs())),
            cf.EPI_STORE_T: (ref, eps * mag),
            cf.EPI_SILU_MUL: (silu * ref2, 1.2 * eps * (mag * ref2.abs() + mag2 * silu.abs() + mag * mag2 * eps) + 2.0 ** -20 * (silu * ref2).abs())}
    for epi, (r, bound) in want.items():
        out = c0.cuda()
        torch.cuda.synchronize()
        as_float = epi in (cf.EPI_STORE_F32, cf.EPI_ADD_F32)
        sess.ctx.op_gemm(A.data_ptr(), W.data_ptr(), W2.data_ptr(), out.data_ptr() if as_float else 0,
                         0 if as_float else out.data_ptr(), M, N, K, epi)
        err = (out.cpu().double() - r).abs()
        assert bool((err <= bound + 1e-30).all()), f"epilogue {epi}: worst {float((err - bound).max())} over its bound"


@pytest.mark.parametrize("hd, hq, hkv, n_ctx, n_new", [
    (128, 4, 2, [1, 15, 16, 17, 33, 130], [1, 16, 17, 2, 31, 5]),          # 16-row blocks
    (64, 8, 8, [3, 129, 40] + [20] * 14, [33, 1, 16] + [1] * 14),          # 32-row blocks
    (128, 8, 1, [31, 128, 65] + [18] * 14, [1, 32, 47] + [2] * 14)])
def test_attention_f32_matches_the_oracle(hd, hq, hkv, n_ctx, n_new):
    """End to end through two layers (1e-4: the stated bound of the float32 model); the pool starts
    as NaN patterns, so a slot past a request's last key must not reach any result."""
    from paper_2604_25080_amd.runtime import Session
    from gpu_util import decode_pages, stack_kv
    shape = ModelShape("f32-2", 2, 256, hq, hkv, hd, 352, 64, 10000.0, 1e-5, "f32")
    ws = WeightSource(shape, 11, cache=True)
    rng = np.random.default_rng(hd + len(n_ctx))
    ids = lambda n: rng.integers(0, shape.vocab, size=n).astype(np.int32)  # noqa: E731
    ctx, new = [ids(n) for n in n_ctx], [ids(n) for n in n_new]
    s = Session(shape, ws, max_batch=len(n_ctx), max_tokens=sum(n_ctx) + sum(n_new), max_positions=256, n_pages=80,
                pool_fill=0xFF)
    for i, (n, m) in enumerate(zip(n_ctx, n_new)):
        s.cache.alloc(1 + i, n + m)
    reqs = [dict(req_id=1 + i, ctx_tokens=ctx[i], new_tokens=new[i]) for i in range(len(n_ctx))]
    logits, _ = s.restore(reqs, [(0, n, shape.n_layers) for n in n_ctx])
    logits = logits.cpu().numpy().astype(np.float64)
    for i, n in enumerate(n_ctx):
        kv_ctx, kv_new, ref = T.full_reference(shape, ws, ctx[i], new[i])
        assert np.abs(logits[i] - ref).max() <= 1e-4
        got = decode_pages(shape, s.read_pages(1 + i, n + n_new[i]), n + n_new[i])
        for a, b in zip(got, stack_kv(shape, kv_ctx, kv_new)):
            assert np.abs(a - b).max() <= 1e-4
    s.close()


@pytest.mark.parametrize("hd, hq, hkv, n_other", [(64, 4, 2, 0), (128, 4, 4, 0), (64, 8, 8, 18), (128, 8, 2, 18)])
def test_attention_f32_a_later_token_that_is_not_finite(hd, hq, hkv, n_other):
    """A token whose embedding is NaN makes its own rows and those behind it NaN; every row before it, and
    every other request, keeps the bits that it has with an ordinary token in that place."""
    from paper_2604_25080_amd.runtime import Session
    from gpu_util import decode_pages
    shape = ModelShape("f32-3", 3, 128, hq, hkv, hd, 160, 64, 10000.0, 1e-5, "f32")

    class Source(WeightSource):
        def storage(self, name, layer=-1):
            w = super().storage(name, layer)
            if name == "embed":
                w[63] = np.nan
            return w

    rng = np.random.default_rng(hd + hq)
    n_ctx, n_new = [40, 53, 21] + [18] * n_other, [20, 35, 17] + [2] * n_other
    ctx, new = ([rng.integers(0, 63, size=n).astype(np.int32) for n in v] for v in (n_ctx, n_new))
    at = {0: 38, 1: 53 + 18}                                   # in a context, in a new turn; request 2 has none
    s = Session(shape, Source(shape, 12), max_batch=len(n_ctx), max_tokens=sum(n_ctx) + sum(n_new), max_positions=128,
                n_pages=4 * len(n_ctx) + 8, pool_fill=0xFF)
    for i, (n, m) in enumerate(zip(n_ctx, n_new)):
        s.cache.alloc(1 + i, n + m)

    def run():
        reqs = [dict(req_id=1 + i, ctx_tokens=ctx[i], new_tokens=new[i]) for i in range(len(n_ctx))]
        logits, _ = s.restore(reqs, [(0, n, shape.n_layers) for n in n_ctx])
        cells = [np.stack(decode_pages(shape, s.read_pages(1 + i, n + m), n + m)) for i, (n, m) in enumerate(zip(n_ctx, n_new))]
        return logits.cpu().numpy().copy(), cells

    clean_logits, clean = run()
    assert np.isfinite(clean_logits).all()
    for i, j in at.items():
        (ctx if j < n_ctx[i] else new)[i][j if j < n_ctx[i] else j - n_ctx[i]] = 63
    logits, cells = run()
    for i in range(len(n_ctx)):
        j = at.get(i, n_ctx[i] + n_new[i])
        assert np.array_equal(cells[i][:, :, :j], clean[i][:, :, :j]), f"request {i}: rows before position {j}"
        assert np.isnan(cells[i][:, 1:, j:]).all()
        assert np.array_equal(logits[i], clean_logits[i]) if i not in at else np.isnan(logits[i]).all()
    s.close()
