"""GPU kernel parity: the MFMA GEMM (all fused epilogues) and the plain FMA
GEMM against the definition (a float64 matmul of the same bf16 inputs), at
sizes that span several tiles with ragged tails."""
import numpy as np
import pytest
import torch

from workloads import SHAPES, WeightSource, bf16_bits, bits_to_f32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sess():
    from paper_2604_25080_amd.runtime import Session
    shape = SHAPES["mini-bf16"].with_layers(1)
    s = Session(shape, WeightSource(shape, 5), max_batch=2, max_tokens=256, max_positions=256, n_pages=8)
    real = s.ctx
    s.ctx = _Synced(real)
    yield s
    s.ctx = real
    s.close()


class _Synced:
    """The library launches on its own streams, which do not order against torch's: operands and
    output buffers made by torch kernels (fills, slices) must be complete before a library call."""

    def __init__(self, ctx):
        self._ctx = ctx

    def op_gemm(self, *a, **k):
        torch.cuda.synchronize()
        return self._ctx.op_gemm(*a, **k)


def dev_bf16(x):
    return torch.from_numpy(bf16_bits(x).view(np.int16)).cuda().view(torch.bfloat16)


def from_bf16(t):
    return bits_to_f32(t.view(torch.int16).cpu().numpy().view(np.uint16).reshape(-1)).reshape(t.shape)


SHAPES_MNK = [(256, 256, 64), (300, 544, 512), (1000, 1408, 512), (129, 96, 1408), (2, 2000, 512),
              (2048, 1280, 1024)]


@pytest.mark.parametrize("impl", [3, 4, 5, 1, 6])
@pytest.mark.parametrize("mnk", SHAPES_MNK + [(4400, 4096, 128)])
def test_gemm_epilogues_match_float64_matmul(sess, impl, mnk):
    import paper_2604_25080_amd as cf
    M, N, K = mnk
    rng = np.random.default_rng(M * 7 + N)
    a = bits_to_f32(bf16_bits(rng.normal(size=(M, K)).astype(np.float32)))
    w = bits_to_f32(bf16_bits((rng.normal(size=(N, K)) * 0.05).astype(np.float32)))
    w2 = bits_to_f32(bf16_bits((rng.normal(size=(N, K)) * 0.05).astype(np.float32)))
    ref = a.astype(np.float64) @ w.astype(np.float64).T
    ref2 = a.astype(np.float64) @ w2.astype(np.float64).T
    A, W, W2 = dev_bf16(a), dev_bf16(w), dev_bf16(w2)
    Cf = torch.zeros(M, N, dtype=torch.float32, device="cuda")
    Dt = torch.zeros(M, N, dtype=torch.bfloat16, device="cuda")
    tol = 1e-4 * np.sqrt(K / 512)

    sess.ctx.op_gemm(A.data_ptr(), W.data_ptr(), 0, Cf.data_ptr(), 0, M, N, K, cf.EPI_STORE_F32, impl)
    assert np.abs(Cf.cpu().numpy() - ref).max() <= tol
    base = torch.from_numpy(rng.normal(size=(M, N)).astype(np.float32)).cuda()
    Cf.copy_(base)
    sess.ctx.op_gemm(A.data_ptr(), W.data_ptr(), 0, Cf.data_ptr(), 0, M, N, K, cf.EPI_ADD_F32, impl)
    assert np.abs(Cf.cpu().numpy() - (ref + base.cpu().numpy())).max() <= tol
    sess.ctx.op_gemm(A.data_ptr(), W.data_ptr(), 0, 0, Dt.data_ptr(), M, N, K, cf.EPI_STORE_T, impl)
    got = from_bf16(Dt)
    assert np.all(np.abs(got - ref) <= np.abs(ref) * 2.0 ** -8 + tol)      # one bf16 rounding
    sess.ctx.op_gemm(A.data_ptr(), W.data_ptr(), W2.data_ptr(), 0, Dt.data_ptr(), M, N, K, cf.EPI_SILU_MUL, impl)
    want = ref / (1.0 + np.exp(-ref)) * ref2
    got = from_bf16(Dt)
    assert np.all(np.abs(got - want) <= np.abs(want) * 2.0 ** -8 + 4 * tol)


# (4352, 4096): 17 x 16 = 272 big tiles = one round of 256 and 16 more: the mixed launch covers a
# 1 x 16 rectangle with 128x128 tiles; (4400, 4104): ragged edges, 18 x 17 = 306 tiles, tail 50
# rounded up to 2 x 25 > 17 columns, so the plain launch; (4660, 4360): 19 x 18 = 342, tail 86 =
# 3 rows x 29 > 18: plain; (8192, 2100): 32 x 9 = 288, tail 32 = 8 rows x 4 columns, ragged N
@pytest.mark.parametrize("mnk", [(300, 544, 512), (129, 4096, 1024), (16, 1280, 8192), (2048, 1280, 1024),
                                 (600, 768, 1408), (4352, 4096, 256), (4400, 4104, 256), (8192, 2100, 128),
                                 (4500, 4096, 128)])
def test_gemm_bits_do_not_depend_on_the_tile_shape(sess, mnk):
    """Every output element is accumulated in the same order along K whatever the block tile
    (256x256, 128x128, 64x64 with its deeper operand pipeline) and whatever else is in the
    launch: hybrid == all-recompute == chunk-by-chunk restores rest on this."""
    import paper_2604_25080_amd as cf
    M, N, K = mnk
    rng = np.random.default_rng(M + N + K)
    A = dev_bf16(rng.normal(size=(M, K)).astype(np.float32))
    W = dev_bf16((rng.normal(size=(N, K)) * 0.05).astype(np.float32))
    outs, impls = [], []
    for impl in (3, 6, 4, 5, 0):
        if impl in (3, 6) and (M < 256 or N < 256 or K % 128):
            continue
        Cf = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        sess.ctx.op_gemm(A.data_ptr(), W.data_ptr(), 0, Cf.data_ptr(), 0, M, N, K, cf.EPI_STORE_F32, impl)
        outs.append(Cf)
        impls.append(impl)
    # a sub-range of the rows on its own gives the same bits for those rows
    lo = M // 3
    Cs = torch.full((M - lo, N), float("nan"), dtype=torch.float32, device="cuda")
    sess.ctx.op_gemm(A[lo:].contiguous().data_ptr(), W.data_ptr(), 0, Cs.data_ptr(), 0, M - lo, N, K,
                     cf.EPI_STORE_F32, 0)
    for o, impl in zip(outs[1:], impls[1:]):
        if not torch.equal(outs[0], o):
            bad = torch.nonzero((outs[0] != o) | torch.isnan(o))
            raise AssertionError(f"impl {impl} differs from impl {impls[0]} in {len(bad)} elements, first at "
                                 f"{bad[0].tolist()}, last at {bad[-1].tolist()}; NaN left: {int(torch.isnan(o).sum())}")
    assert torch.equal(outs[0][lo:], Cs)


@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 65])
@pytest.mark.parametrize("nk", [(96, 64), (130, 192), (1000, 1408), (64, 72), (33, 688), (2000, 712)])
def test_gemm_few_rows_and_ragged_k(sess, rows, nk):
    """Row counts at the edges of the few-row kernel, K of one step, of ragged groups of steps and
    ending inside a step (72, 688, 712: whole 16-byte vectors).  The rows must come out with the bits
    that they get inside a taller launch; 2^-24 per term against float64; the operands are followed by
    NaN, which a read past a row's end would let in."""
    import paper_2604_25080_amd as cf
    N, K = nk
    M = 700
    g = torch.Generator().manual_seed(rows * 7 + N + K)
    a, w, w2 = (torch.full((r * K + 64,), float("nan")).bfloat16() for r in (M, N, N))
    for t, r, std in ((a, M, 1.0), (w, N, 0.05), (w2, N, 0.05)):
        t[:r * K] = (torch.randn(r * K, generator=g) * std).bfloat16()
    A, W, W2 = a.cuda(), w.cuda(), w2.cuda()
    few = a.clone()
    few[rows * K:] = float("nan")
    Few = few.cuda()
    x, y, y2 = a[:rows * K].view(rows, K).double(), w[:N * K].view(N, K).double(), w2[:N * K].view(N, K).double()
    ref, ref2 = x @ y.t(), x @ y2.t()
    for epi in (cf.EPI_STORE_F32, cf.EPI_STORE_T, cf.EPI_SILU_MUL):
        dt = torch.float32 if epi == cf.EPI_STORE_F32 else torch.bfloat16
        out, tall = torch.zeros(rows, N, dtype=dt, device="cuda"), torch.zeros(M, N, dtype=dt, device="cuda")
        for src, dst, m in ((Few, out, rows), (A, tall, M)):
            p = dst.data_ptr()
            sess.ctx.op_gemm(src.data_ptr(), W.data_ptr(), W2.data_ptr(), p if dt == torch.float32 else 0,
                             0 if dt == torch.float32 else p, m, N, K, epi, 0)
        assert torch.equal(out, tall[:rows])
        if epi == cf.EPI_STORE_F32:
            err, bound = (out.cpu().double() - ref).abs(), K * 2.0 ** -24 * (x.abs() @ y.abs().t())
        else:
            r = ref if epi == cf.EPI_STORE_T else ref * torch.sigmoid(ref) * ref2
            err, bound = (out.cpu().double() - r).abs(), 2.0 ** -8 * r.abs() + 1e-5
        assert bool((err <= bound).all())


def _placed(x, rows, K):
    """The first rows of x [M, K] on the device, NaN behind them."""
    t = torch.full((rows * K + 64,), float("nan")).bfloat16()
    t[:rows * K] = x[:rows].reshape(-1)
    return t.cuda()


@pytest.mark.parametrize("K", [72, 712])
def test_gemm_ragged_k_on_the_128_tile(sess, K):
    """1700 x 2000 is more than three 64-wide tiles per CU: the 128x128 tile, with a last K-step that is partly
    past the rows' end.  2^-24 per term against float64, and the bits that 65 rows get on the 64 tile."""
    import paper_2604_25080_amd as cf
    M, N, few = 1700, 2000, 65
    g = torch.Generator().manual_seed(K)
    x, y, y2 = ((torch.randn(r, K, generator=g) * std).bfloat16() for r, std in ((M, 1.0), (N, 0.05), (N, 0.05)))
    A, Few, W, W2 = _placed(x, M, K), _placed(x, few, K), _placed(y, N, K), _placed(y2, N, K)
    x, y, y2 = x.double(), y.double(), y2.double()
    ref, ref2 = x @ y.t(), x @ y2.t()
    for epi in (cf.EPI_STORE_F32, cf.EPI_SILU_MUL):
        as_float = epi == cf.EPI_STORE_F32
        outs = []
        for src, m in ((A, M), (Few, few)):
            out = torch.zeros(m, N, dtype=torch.float32 if as_float else torch.bfloat16, device="cuda")
            p = out.data_ptr()
            sess.ctx.op_gemm(src.data_ptr(), W.data_ptr(), W2.data_ptr(), p if as_float else 0, 0 if as_float else p, m, N, K, epi)
            outs.append(out)
        assert torch.equal(outs[0][:few], outs[1])
        r = ref if as_float else ref * torch.sigmoid(ref) * ref2
        bound = K * 2.0 ** -24 * (x.abs() @ y.abs().t()) if as_float else 2.0 ** -8 * r.abs() + 1e-5
        assert bool(((outs[0].cpu().double() - r).abs() <= bound).all())


# 16 tile columns: 336, 368 and 384 big tiles, 80, 112 and 128 of them past the first round
@pytest.mark.parametrize("tiles_m, K", [(21, 1024), (23, 1152), (24, 2048)])
def test_gemm_quartered_tail_over_long_k(sess, tiles_m, K):
    """The tail's 128x128 tiles with more K-steps than their ring holds, up to half a round of them, ragged in M
    (and N): the bits of the plain launch of big tiles, and 2^-24 per term against float64."""
    import paper_2604_25080_amd as cf
    M = tiles_m * 256 - 5
    g = torch.Generator("cuda").manual_seed(M + K)
    mat = lambda r, std: (torch.randn(r, K, generator=g, device="cuda") * std).bfloat16()  # noqa: E731
    a = mat(M, 1.0)
    for epi, N in ((cf.EPI_STORE_F32, 4090), (cf.EPI_STORE_T, 4096), (cf.EPI_SILU_MUL, 2044)):
        w, w2 = mat(N, 0.05), mat(N, 0.05)
        outs = []
        for impl in (3, 6):
            out = torch.full((M, N), float("nan"), dtype=torch.float32 if epi == cf.EPI_STORE_F32 else torch.bfloat16, device="cuda")
            p, as_float = out.data_ptr(), epi == cf.EPI_STORE_F32
            sess.ctx.op_gemm(a.data_ptr(), w.data_ptr(), w2.data_ptr(), p if as_float else 0, 0 if as_float else p, M, N, K, epi, impl)
            outs.append(out)
        assert torch.equal(outs[0], outs[1])
        if epi == cf.EPI_STORE_F32:
            x, y = a.double(), w.double()
            assert bool(((outs[1].double() - x @ y.t()).abs() <= K * 2.0 ** -24 * (x.abs() @ y.abs().t())).all())


@pytest.mark.parametrize("at_a, at_w", [(2, 0), (0, 6), (1, 0), (0, 3)])
def test_gemm_operands_that_start_inside_a_larger_buffer(sess, at_a, at_w):
    """Whole-dword starts are loaded straight to LDS, odd elements through registers; 2^-24 per term."""
    import paper_2604_25080_amd as cf
    M, N, K = 130, 200, 192
    g = torch.Generator().manual_seed(at_a + 10 * at_w)
    a, w = (torch.randn(r * K + 8, generator=g).bfloat16() for r in (M, N))
    A, W, Cf = a.cuda(), w.cuda(), torch.zeros(M, N, device="cuda")
    sess.ctx.op_gemm(A.data_ptr() + 2 * at_a, W.data_ptr() + 2 * at_w, 0, Cf.data_ptr(), 0, M, N, K, cf.EPI_STORE_F32, 0)
    x, y = a[at_a:at_a + M * K].view(M, K).double(), w[at_w:at_w + N * K].view(N, K).double()
    assert bool(((Cf.cpu().double() - x @ y.t()).abs() <= K * 2.0 ** -24 * (x.abs() @ y.abs().t())).all())


@pytest.mark.parametrize("mnk", [(1, 96, 64), (16, 1280, 1024), (33, 130, 72), (300, 544, 512), (700, 2001, 712),
                                 (1700, 2000, 712), (2900, 3075, 256)])
def test_gemm_operands_at_odd_elements_give_the_same_bits(sess, mnk):
    """Every tile (forced where the call takes that: K of whole steps), float and 16-bit outputs, operands
    followed by NaN; against the same operands on 16-byte boundaries."""
    import paper_2604_25080_amd as cf
    M, N, K = mnk
    g = torch.Generator().manual_seed(M + N + K)
    parts = [(torch.randn(r * K, generator=g) * std).bfloat16() for r, std in ((M, 1.0), (N, 0.05), (N, 0.05))]

    def placed(x, at):
        t = torch.full((x.numel() + 64,), float("nan")).bfloat16()
        t[at:at + x.numel()] = x
        return t.cuda()[at:]

    even, odd = [placed(x, 0) for x in parts], [placed(x, at) for x, at in zip(parts, (1, 3, 7))]
    base = torch.randn(M, N, generator=g)
    for epi in (cf.EPI_STORE_F32, cf.EPI_ADD_F32, cf.EPI_STORE_T, cf.EPI_SILU_MUL):
        for impl in (0, 3, 4, 5) if K % 64 == 0 else (0,):
            outs = []
            for a, w, w2 in (even, odd, (even[0], odd[1], even[2]), (odd[0], even[1], odd[2])):
                out = base.cuda() if epi in (cf.EPI_STORE_F32, cf.EPI_ADD_F32) else base.bfloat16().cuda()
                p, as_float = out.data_ptr(), out.dtype == torch.float32
                sess.ctx.op_gemm(a.data_ptr(), w.data_ptr(), w2.data_ptr(), p if as_float else 0, 0 if as_float else p,
                                 M, N, K, epi, impl)
                outs.append(out)
            assert not bool(torch.isnan(outs[0].float()).any())
            assert all(torch.equal(outs[0], o) for o in outs[1:]), f"epilogue {epi}, impl {impl}"


@pytest.mark.parametrize("impl", [0, 3, 4])
def test_gemm_rows_that_pass_the_32_bit_offsets(sess, impl):
    """256 rows of 2^23 elements are 2^32 bytes, more than a tile's 32-bit offsets reach.  Few entries are not
    zero, so the sums are whole numbers and exact."""
    import paper_2604_25080_amd as cf
    M, N, K = 256, 256, 1 << 23
    A, W = (torch.zeros(r, K, dtype=torch.bfloat16, device="cuda") for r in (M, N))
    cols = [0, 7, 64, 4099, (1 << 22) - 1, 1 << 22, K - 65, K - 1]
    g = torch.Generator().manual_seed(3)
    a, w = (torch.randint(-4, 5, (r, len(cols)), generator=g).float() for r in (M, N))
    A[:, cols], W[:, cols] = a.bfloat16().cuda(), w.bfloat16().cuda()
    Cf = torch.full((M, N), float("nan"), device="cuda")
    sess.ctx.op_gemm(A.data_ptr(), W.data_ptr(), 0, Cf.data_ptr(), 0, M, N, K, cf.EPI_STORE_F32, impl)
    assert torch.equal(Cf.cpu(), a @ w.t())


def test_gemm_mfma_refuses_what_it_cannot_tile(sess):
    import paper_2604_25080_amd as cf
    A = torch.zeros(64, 40, dtype=torch.bfloat16, device="cuda")
    Cf = torch.zeros(64, 64, dtype=torch.float32, device="cuda")
    with pytest.raises(cf.CfError) as e:
        sess.ctx.op_gemm(A.data_ptr(), A.data_ptr(), 0, Cf.data_ptr(), 0, 64, 64, 40, cf.EPI_STORE_F32, 2)
    assert e.value.status == cf.CF_ERR_UNSUPPORTED
    sess.ctx.op_gemm(A.data_ptr(), A.data_ptr(), 0, Cf.data_ptr(), 0, 64, 64, 40, cf.EPI_STORE_F32, 0)
