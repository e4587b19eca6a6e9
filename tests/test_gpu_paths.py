"""Kernel variants at the sizes where their tiles, slices and row tails end,
against the float64 oracle.  Bounds: the float32 sums of exact products (bf16
values multiply exactly in float32) stay within the norm and gradient guards
of tolerances.py; float32 inputs within its gates."""
import numpy as np
import pytest
import torch

import oracle
from tolerances import GRAD_GATE, GRAD_GUARD_EXACT, GRAD_GUARD_ROUNDED, NORM_GATE, NORM_GUARD  # noqa: F401

pytestmark = pytest.mark.gpu
DEV = "cuda"
BF, F32 = torch.bfloat16, torch.float32


@pytest.fixture(scope="module")
def bk():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2210_00038_amd as m
    return m


def _rel(x, ref):
    x, ref = np.asarray(x, np.float64), np.asarray(ref, np.float64)
    return np.max(np.abs(x - ref) / np.maximum(np.abs(ref), 1e-300)) if ref.size else 0.0


def _frob(x, ref):
    x, ref = np.asarray(x, np.float64), np.asarray(ref, np.float64)
    n = np.linalg.norm(ref)
    return np.linalg.norm(x - ref) / n if n > 0 else np.linalg.norm(x)


def _norm_bound(dtype):
    return NORM_GATE["f32"] if dtype == F32 else NORM_GUARD


def _draw(B, T, d, dtype, gen, scale=1.0, offset=0):
    """[B, T, d] values; offset: elements by which the first one misses 16-byte alignment."""
    buf = torch.full((B * T * d + offset + 16,), float("nan"), dtype=dtype, device=DEV)
    x = buf[offset:offset + B * T * d].view(B, T, d)
    v = (torch.randn(B, T, d, generator=gen) * scale).to(dtype)
    x.copy_(v)
    return x, v


# One 128-row block or several, rows of any alignment or of 16-byte multiples,
# few enough (sample, pair) workgroups that the rows are cut into column slices.
@pytest.mark.parametrize("B,T,d,p,dtype,off", [
    (2, 100, 1031, 4099, BF, 0),     # odd rows, slices with a ragged last chunk
    (1, 128, 768, 5000, BF, 0),      # 16-byte rows, slices
    (2, 130, 2051, 1025, F32, 0),    # two row blocks, odd float32 rows, slices
    (2, 200, 1000, 1032, BF, 3),     # 16-byte row lengths, misaligned base
    (3, 100, 7, 3, BF, 0),           # rows shorter than 16 bytes
    (3, 70, 3, 41, F32, 0),
    (2, 65, 8, 9, BF, 0),            # rows of exactly one piece, and one element more
    (300, 66, 13, 71, BF, 0),        # enough workgroups: no slices
])
def test_ghost_rows_and_column_slices(bk, B, T, d, p, dtype, off):
    gen = torch.Generator().manual_seed(B * 100 + T + d)
    a, ah = _draw(B, T, d, dtype, gen, 1.0, off)
    g, gh = _draw(B, T, p, dtype, gen, 1e-2, off)
    a[B - 1].zero_()
    ah[B - 1] = 0
    ref = oracle.linear_norm_sq(ah, gh)
    out = bk.bk_ghost_norm(a, g)
    assert torch.equal(out, bk.bk_ghost_norm(a, g))
    out = out.cpu().numpy()
    assert out[B - 1] == 0.0 and _rel(out[:B - 1], ref[:B - 1]) <= _norm_bound(dtype)
    # in a stack with a bias (its sums run apart when the rows are sliced)
    Pb, norm = torch.empty(B, p, device=DEV), torch.empty(2, B, device=DEV)
    arr = bk.make_layers([{"x": a, "g": g, "bias": True, "Pb": Pb}, {"x": a, "g": g}])
    bk.bk_layer_norms(arr, 2, bk.BK_BF16 if dtype == BF else bk.BK_F32, B, norm)
    sb = oracle.bias_sums(gh)
    got = norm.cpu().numpy()
    assert _frob(Pb.cpu().numpy(), sb) <= 1e-5
    assert _rel(got[0], ref + (sb ** 2).sum(1)) <= _norm_bound(dtype)
    assert _rel(got[1][:B - 1], ref[:B - 1]) <= _norm_bound(dtype)


# bf16 rows of any alignment on the 256 x 128 tiles: ragged last pieces of
# either operand, row counts around the 64-row stage, several tiles.
@pytest.mark.parametrize("B,T,d,p,off", [
    (2, 40, 8, 9, 0),          # one piece per row, one element more
    (3, 64, 257, 131, 0),      # one column past a tile on both sides, whole stages
    (3, 65, 255, 127, 0),      # one column short of a tile, one row past a stage
    (5, 13, 1000, 15, 0),      # several samples per stage
    (2, 130, 264, 136, 1),     # 16-byte row lengths, misaligned base
    (130, 1, 300, 10, 0),      # one token a sample
    (2, 1, 300, 131, 0),       # two rows in all (the element-load kernel), and three
    (3, 1, 300, 131, 0),
    (3, 65, 300, 2, 0),        # rows of fewer than 8 elements: two, one
    (4, 70, 1, 131, 0),
    (3, 100, 7, 3, 1),         # both sides, the batch ends inside a piece
    (8, 1, 1, 72, 0),          # one piece in all
])
def test_gemm_rows_of_any_alignment(bk, B, T, d, p, off):
    gen = torch.Generator().manual_seed(B + 10 * T + d)
    a, ah = _draw(B, T, d, BF, gen, 1.0, off)
    g, gh = _draw(B, T, p, BF, gen, 1e-2, off)
    # what lies around the rows must not reach the results
    C = torch.rand(B, generator=gen) + 0.1
    C[B // 2] = 0.0
    G = bk.bk_weighted_grad(a, g, C.to(DEV))
    assert _frob(G.cpu().numpy(), oracle.weighted_grad(ah, gh, C)) <= GRAD_GUARD_ROUNDED
    C2 = torch.exp2(torch.randint(-3, 4, (B,), generator=gen).float())       # exact in bf16
    G = bk.bk_weighted_grad(a, g, C2.to(DEV))
    assert _frob(G.cpu().numpy(), oracle.weighted_grad(ah, gh, C2)) <= GRAD_GUARD_EXACT
    norm, P = bk.bk_per_sample_grads(a, g)
    assert torch.equal(norm, bk.bk_inst_norm(a, g))
    assert _rel(norm.cpu().numpy(), oracle.linear_norm_sq(ah, gh)) <= NORM_GUARD
    assert _frob(P.cpu().numpy(), oracle.per_sample_grads(ah, gh)) <= GRAD_GUARD_EXACT


# Few tokens: 32 / T whole samples to a 32-row block up to T = 16, one sample
# to a 32- or 64-row block up to T = 64; the last block partly filled, rows of
# every alignment, one chunk of columns and several, a bias in the same pass.
@pytest.mark.parametrize("dtype", [BF, F32])
@pytest.mark.parametrize("B,T,d,p,off", [
    (1, 1, 64, 40, 0),         # one sample, one token
    (70, 1, 768, 1000, 0),     # 32 samples a block, six in the last one
    (33, 1, 591, 675, 0),      # odd rows
    (5, 2, 7, 1300, 0),        # rows shorter than 16 bytes beside long ones
    (9, 5, 300, 260, 1),       # 6 samples a block (30 rows), misaligned base
    (7, 16, 256, 264, 0),      # two samples a block
    (3, 17, 520, 72, 0),       # one sample a block from here on
    (4, 32, 100, 257, 0),
    (3, 33, 264, 129, 0),      # two 32-row blocks, one row in the second
    (2, 64, 1032, 1000, 0),
    (2, 50, 4000, 5000, 0),    # long rows, few workgroups: column slices of the pair kernel
])
def test_ghost_few_tokens(bk, B, T, d, p, off, dtype):
    gen = torch.Generator().manual_seed(B * 100 + T + d)
    a, ah = _draw(B, T, d, dtype, gen, 1.0, off)
    g, gh = _draw(B, T, p, dtype, gen, 1e-2, off)
    if B > 1:
        a[B - 1].zero_()
        ah[B - 1] = 0
    ref = oracle.linear_norm_sq(ah, gh)
    out = bk.bk_ghost_norm(a, g)
    assert torch.equal(out, bk.bk_ghost_norm(a, g))
    out = out.cpu().numpy()
    n = max(1, B - 1)
    assert _rel(out[:n], ref[:n]) <= _norm_bound(dtype) and (B == 1 or out[B - 1] == 0.0)
    if not oracle.use_ghost(T, d, p):
        return
    Pb, norm = torch.full((B, p), float("nan"), device=DEV), torch.empty(2, B, device=DEV)
    arr = bk.make_layers([{"x": a, "g": g, "bias": True, "Pb": Pb}, {"x": a, "g": g}])
    bk.bk_layer_norms(arr, 2, bk.BK_BF16 if dtype == BF else bk.BK_F32, B, norm)
    sb = oracle.bias_sums(gh)
    got = norm.cpu().numpy()
    assert _frob(Pb.cpu().numpy(), sb) <= 1e-6
    assert _rel(got[0], ref + (sb ** 2).sum(1)) <= _norm_bound(dtype)
    assert _rel(got[1][:n], ref[:n]) <= _norm_bound(dtype)


# Samples of few and of more tokens in one small call: the shorter ones run in
# the launch of the longer, one sample to a workgroup, bias sums too.
@pytest.mark.parametrize("dtype,B,Ts,d,p", [
    (BF, 3, (1, 16, 40), 200, 136), (BF, 7, (5, 33), 130, 1000), (F32, 2, (17, 64), 68, 200), (F32, 3, (4, 50, 80, 120), 257, 260)])
def test_ghost_few_and_more_tokens_together(bk, dtype, B, Ts, d, p):
    gen = torch.Generator().manual_seed(B + d)
    xs = [(_draw(B, T, d, dtype, gen), _draw(B, T, p, dtype, gen, 1e-2)) for T in Ts]
    assert all(oracle.use_ghost(T, d, p) for T in Ts)
    Pb, norm = torch.full((len(Ts), B, p), float("nan"), device=DEV), torch.empty(len(Ts), B, device=DEV)
    arr = bk.make_layers([{"x": a, "g": g, "bias": True, "Pb": Pb[i]} for i, ((a, _), (g, _)) in enumerate(xs)])
    bk.bk_layer_norms(arr, len(Ts), bk.BK_BF16 if dtype == BF else bk.BK_F32, B, norm)
    for i, ((_, ah), (_, gh)) in enumerate(xs):
        sb = oracle.bias_sums(gh)
        assert _frob(Pb[i].cpu().numpy(), sb) <= 1e-6
        assert _rel(norm[i].cpu().numpy(), oracle.linear_norm_sq(ah, gh) + (sb ** 2).sum(1)) <= _norm_bound(dtype)


# Every way the few-token kernel's loop over chunks can end (a's and g's of one
# chunk, an even and an odd number) and the whole-sample kernel's, without a
# bias: right, and the same bits from every run.
@pytest.mark.parametrize("dtype,T,na,ng", [
    (dt, T, na, ng) for dt, T in ((BF, 1), (F32, 1), (BF, 37), (F32, 37), (BF, 150), (BF, 256))
    for na, ng in ((1, 1), (2, 1), (1, 2), (2, 2), (3, 1), (2, 3))])
def test_ghost_chunk_counts(bk, dtype, T, na, ng):
    chunk = 64 if T > 64 else (256 if T <= 32 else 128) // (1 if dtype == BF else 2)
    B, d, p = (1151, chunk * na - 3, chunk * ng - 5) if T == 1 else (70, chunk * na, chunk * ng - 8)
    gen = torch.Generator().manual_seed(T + 10 * na + ng)
    a, ah = _draw(B, T, d, dtype, gen)
    g, gh = _draw(B, T, p, dtype, gen, 1e-2)
    out = bk.bk_ghost_norm(a, g)
    assert _rel(out.cpu().numpy(), oracle.linear_norm_sq(ah, gh)) <= _norm_bound(dtype)
    for _ in range(50):
        assert torch.equal(out, bk.bk_ghost_norm(a, g))


# Short vectors over at least 16 samples: 16 interleaved runs of samples per
# element (64 elements a workgroup); longer vectors or fewer samples: one run.
@pytest.mark.parametrize("B,n,accum", [
    (16, 64, False), (17, 63, False), (1000, 1000, True), (33, 1, False), (15, 64, True), (16, 65536, False),
    (16, 65540, True)])
def test_weighted_sum_runs(bk, B, n, accum):
    gen = torch.Generator().manual_seed(B + n)
    P = torch.randn(B, n, generator=gen)
    C = torch.rand(B, generator=gen) + 0.05
    G = bk.bk_weighted_sum(P.to(DEV), C.to(DEV))
    # B float32 products and additions: at most (B + 1) roundings of 2^-24 each
    assert _frob(G.cpu().numpy(), oracle.weighted_sum(P.numpy(), C.numpy())) <= (B + 1) * 2.0 ** -24
    if accum and n <= 1024:           # as the bias of a layer that accumulates
        x = torch.zeros(B, 1, n, dtype=BF, device=DEV)
        Gb = torch.randn(n, generator=gen).to(DEV)
        want = Gb + G
        arr = bk.make_layers([{"x": x, "g": x, "G": torch.zeros(n, n, device=DEV), "bias": True, "Gb": Gb,
                               "Pb": P.to(DEV), "accumulate": True}])
        bk.bk_weighted_grads(arr, 1, C.to(DEV), bk.BK_BF16, B)
        assert torch.equal(Gb, want)


# Layers of T < 64 and others whose samples do not pad to 16-row steps.  `flat`:
# the 256 x 256 DMA tiles over the flat rows of the batch, weights on g's
# fragments (T > 64, or at least 4096 rows): several samples per 32-row stage and
# per 16-row step, last stages of every kind, zero weights; their single layers
# of few tiles run in K slices, which the workspace shows.  Else the 256 x 128
# tiles, unsliced.
@pytest.mark.parametrize("B,T,d,p,flat", [
    (1, 1, 256, 256, False),       # one row
    (33, 1, 264, 136, False),      # one row past a stage
    (3, 16, 128, 72, False),       # 48 rows
    (5, 37, 512, 264, False),      # samples across stages, ragged tiles
    (2, 63, 80, 520, False),
    (9, 13, 300, 200, False),      # odd rows
    (80, 20, 256, 512, False),
    (1100, 1, 768, 200, False),
    (6, 65, 264, 264, False),      # flat, but too few stages for slices
    (4096, 1, 768, 200, True),     # a sample per row, the fullest weight table
    (206, 20, 256, 512, True),     # 4120 rows: samples of 20 across steps of 16
    (316, 13, 304, 200, True),     # 4108: a last stage of one step
    (111, 37, 512, 264, True),     # 4107 rows, ragged tiles
    (70, 63, 264, 136, True),      # the longest T
    (40, 70, 264, 264, True),      # T > 64, padding over 1/8
])
def test_flat_weighted_grad(bk, B, T, d, p, flat):
    assert (bk.bk_workspace_size(bk.BK_OP_WEIGHTED_GRAD, bk.BK_BF16, B, T, d, p) > 0) == flat
    gen = torch.Generator().manual_seed(B + T + d)
    a, ah = _draw(B, T, d, BF, gen)
    g, gh = _draw(B, T, p, BF, gen, 1e-2)
    C = torch.rand(B, generator=gen) + 0.1
    C[B // 2] = 0.0
    G = bk.bk_weighted_grad(a, g, C.to(DEV))
    ref = oracle.weighted_grad(ah, gh, C)
    assert _frob(G.cpu().numpy(), ref) <= GRAD_GUARD_ROUNDED
    C2 = torch.exp2(torch.randint(-3, 4, (B,), generator=gen).float())       # exact in bf16
    G2 = bk.bk_weighted_grad(a, g, C2.to(DEV))
    assert _frob(G2.cpu().numpy(), oracle.weighted_grad(ah, gh, C2)) <= GRAD_GUARD_EXACT
    # two layers in one launch, one of them adding to its gradient
    G0 = torch.randn(d, p, generator=gen).to(DEV)
    Ga, Gw = G0.clone(), torch.empty(d, p, device=DEV)
    arr = bk.make_layers([{"x": a, "g": g, "G": Ga, "accumulate": True}, {"x": a, "g": g, "G": Gw}])
    bk.bk_weighted_grads(arr, 2, C.to(DEV), bk.BK_BF16, B)
    assert torch.equal(Ga, G0 + Gw) and _frob(Gw.cpu().numpy(), ref) <= GRAD_GUARD_ROUNDED


# The flat form by its tiles: 16 x 9 = 144 of 256 x 256 from 512 rows on (whole
# tiles, no slices), one layer narrow (256 x 128 tiles in slices, beside them).
@pytest.mark.parametrize("B,T", [(28, 37), (512, 1), (79, 13)])
def test_flat_weighted_grad_many_tiles(bk, B, T):
    gen = torch.Generator().manual_seed(B)
    a, ah = _draw(B, T, 768, BF, gen)
    g, gh = _draw(B, T, 768, BF, gen, 1e-2)
    n, nh = _draw(B, T, 32, BF, gen, 1e-2)
    C = torch.rand(B, generator=gen) + 0.1
    Gs = torch.full((16, 768, 768), float("nan"), device=DEV)
    Gn = torch.empty(768, 32, device=DEV)
    arr = bk.make_layers([{"x": a, "g": g, "G": Gs[i]} for i in range(16)] + [{"x": a, "g": n, "G": Gn}])
    bk.bk_weighted_grads(arr, 17, C.to(DEV), bk.BK_BF16, B)
    ref = oracle.weighted_grad(ah, gh, C)
    assert _frob(Gs[0].cpu().numpy(), ref) <= GRAD_GUARD_ROUNDED
    assert all(torch.equal(Gs[0], Gs[i]) for i in range(1, 16))
    assert _frob(Gn.cpu().numpy(), oracle.weighted_grad(ah, nh, C)) <= GRAD_GUARD_ROUNDED


# More samples than the 256 x 256 kernels' weight table: 256 x 128 tiles in K
# slices, which begin and end inside samples.
@pytest.mark.parametrize("B,T,d,p", [
    (4097, 64, 72, 80),      # one tile, hundreds of slices of whole samples
    (4200, 3, 264, 136),     # 2 x 2 tiles, samples across stages and slices
    (4100, 67, 72, 264),
    (20000, 1, 304, 72),     # one token a sample
])
def test_weighted_grad_past_the_weight_table(bk, B, T, d, p):
    assert bk.bk_workspace_size(bk.BK_OP_WEIGHTED_GRAD, bk.BK_BF16, B, T, d, p) > 0
    gen = torch.Generator().manual_seed(B + T)
    a, ah = _draw(B, T, d, BF, gen)
    g, gh = _draw(B, T, p, BF, gen, 1e-2)
    C = torch.rand(B, generator=gen) + 0.1
    C[B // 2] = 0.0
    G = bk.bk_weighted_grad(a, g, C.to(DEV))
    assert torch.equal(G, bk.bk_weighted_grad(a, g, C.to(DEV)))
    assert _frob(G.cpu().numpy(), oracle.weighted_grad(ah, gh, C)) <= GRAD_GUARD_ROUNDED
    C2 = torch.exp2(torch.randint(-3, 4, (B,), generator=gen).float())       # exact in bf16
    G2 = bk.bk_weighted_grad(a, g, C2.to(DEV))
    assert _frob(G2.cpu().numpy(), oracle.weighted_grad(ah, gh, C2)) <= GRAD_GUARD_EXACT
    G0 = torch.randn(d, p, generator=gen).to(DEV)
    Ga = G0.clone()
    arr = bk.make_layers([{"x": a, "g": g, "G": Ga, "accumulate": True}])
    bk.bk_weighted_grads(arr, 1, C.to(DEV), bk.BK_BF16, B)
    assert torch.equal(Ga, G0 + G)


# The fp32 GEMM: 128 x 128 tiles, 16-row stages, rows of 16-byte multiples and
# of any length, K slices, accumulation, per-sample gradients (calls of few rows
# on the register-transposing kernel; next to the longer layer below, not).
@pytest.mark.parametrize("B,T,d,p,off", [
    (1, 1, 4, 4, 0),           # one row, one piece
    (3, 5, 128, 132, 0),       # 15 rows; one piece past a tile
    (2, 8, 127, 129, 0),       # 16 rows of odd length
    (17, 1, 300, 10, 0),       # one row past a stage, a sample a row
    (4, 64, 256, 384, 0),      # whole tiles, two K slices
    (40, 33, 132, 260, 0),     # many slices, ragged
    (6, 50, 64, 200, 1),       # misaligned base
    (5, 100, 1, 77, 0),        # one column
    (2, 1030, 136, 24, 0),     # long samples: per-sample gradients in K slices too
    (3, 32, 264, 200, 0),      # the most rows of few tiles on the register-transposing kernel,
    (97, 1, 264, 200, 0),      # and one more
    (1, 65, 131, 71, 0),       # the same of odd rows
])
def test_f32_gemm(bk, B, T, d, p, off):
    gen = torch.Generator().manual_seed(B + T + d + p)
    a, ah = _draw(B, T, d, F32, gen, 1.0, off)
    g, gh = _draw(B, T, p, F32, gen, 1e-2, off)
    C = torch.rand(B, generator=gen) + 0.1
    C[B // 2] = 0.0
    G = bk.bk_weighted_grad(a, g, C.to(DEV))
    ref = oracle.weighted_grad(ah, gh, C)
    # random products: sqrt(rows) roundings of the running sum, 2^-24 each
    bound = 4 * np.sqrt(B * T) * 2.0 ** -24 + 2.0 ** -23
    assert _frob(G.cpu().numpy(), ref) <= min(bound, GRAD_GATE["f32"])
    G0 = torch.randn(d, p, generator=gen).to(DEV)
    Ga = G0.clone()
    arr = bk.make_layers([{"x": a, "g": g, "G": Ga, "accumulate": True}])
    bk.bk_weighted_grads(arr, 1, C.to(DEV), bk.BK_F32, B)
    assert torch.equal(Ga, G0 + G)
    norm, P = bk.bk_per_sample_grads(a, g)
    assert torch.equal(norm, bk.bk_inst_norm(a, g))
    assert _rel(norm.cpu().numpy(), oracle.linear_norm_sq(ah, gh)) <= NORM_GATE["f32"]
    assert _frob(P.cpu().numpy(), oracle.per_sample_grads(ah, gh)) <= bound
    # next to a layer of many more rows, which takes slices of its own
    x, xh = _draw(B, 40 * T, 24, F32, gen)
    Gs = [torch.empty(d, p, device=DEV), torch.empty(24, 24, device=DEV)]
    arr = bk.make_layers([{"x": a, "g": g, "G": Gs[0]}, {"x": x, "g": x, "G": Gs[1]}])
    bk.bk_weighted_grads(arr, 2, C.to(DEV), bk.BK_F32, B)
    assert _frob(Gs[0].cpu().numpy(), ref) <= min(bound, GRAD_GATE["f32"])
    assert _frob(Gs[1].cpu().numpy(), oracle.weighted_grad(xh, xh, C)) <= GRAD_GATE["f32"]


# 128 < T <= 256 in a launch of at least 512 (layer, sample) workgroups: the
# whole-sample kernel forms the bias sums too (chunks of 64 columns, rows past T
# zero, one chunk and several).
@pytest.mark.parametrize("B,T,d,p", [(3, 129, 264, 200), (2, 197, 512, 264), (2, 256, 1280, 136)])
def test_bias_in_whole_sample_ghost(bk, B, T, d, p):
    gen = torch.Generator().manual_seed(B + T + p)
    a, ah = _draw(B, T, d, BF, gen)
    g, gh = _draw(B, T, p, BF, gen, 1e-2)
    assert oracle.use_ghost(T, d, p)
    k = -(-512 // B)
    Pb, norm = torch.full((2, B, p), float("nan"), device=DEV), torch.empty(k + 1, B, device=DEV)
    specs = [{"x": a, "g": g, "bias": i < 2, "Pb": Pb[i] if i < 2 else None} for i in range(k + 1)]
    bk.bk_layer_norms(bk.make_layers(specs), k + 1, bk.BK_BF16, B, norm)
    ref, sb = oracle.linear_norm_sq(ah, gh), oracle.bias_sums(gh)
    got = norm.cpu().numpy()
    for i in range(2):
        assert _frob(Pb[i].cpu().numpy(), sb) <= 1e-6
        assert _rel(got[i], ref + (sb ** 2).sum(1)) <= NORM_GUARD
    assert _rel(got[2], ref) <= NORM_GUARD and torch.equal(norm[2], norm[k])


# fp32 samples of 64 < T <= 128: three or four 32-row blocks, one chunk of 64
# columns and several, ragged and short rows, a bias in the same pass.
@pytest.mark.parametrize("B,T,d,p,off", [
    (3, 65, 264, 130, 0), (2, 96, 64, 203, 0), (2, 97, 1000, 63, 0), (4, 128, 516, 1030, 0), (2, 100, 3, 700, 0),
    (3, 128, 256, 192, 1)])
def test_f32_ghost_whole_sample(bk, B, T, d, p, off):
    gen = torch.Generator().manual_seed(B + T + d)
    a, ah = _draw(B, T, d, F32, gen, 1.0, off)
    g, gh = _draw(B, T, p, F32, gen, 1e-2, off)
    a[B - 1].zero_()
    ah[B - 1] = 0
    ref = oracle.linear_norm_sq(ah, gh)
    out = bk.bk_ghost_norm(a, g)
    assert torch.equal(out, bk.bk_ghost_norm(a, g)) and out[B - 1].item() == 0.0
    assert _rel(out.cpu().numpy()[:B - 1], ref[:B - 1]) <= NORM_GATE["f32"]
    if not oracle.use_ghost(T, d, p):
        return
    Pb, norm = torch.full((B, p), float("nan"), device=DEV), torch.empty(2, B, device=DEV)
    arr = bk.make_layers([{"x": a, "g": g, "bias": True, "Pb": Pb}, {"x": a, "g": g}])
    bk.bk_layer_norms(arr, 2, bk.BK_F32, B, norm)
    sb = oracle.bias_sums(gh)
    assert _frob(Pb.cpu().numpy(), sb) <= 1e-6 and torch.equal(norm[1], out)
    assert _rel(norm[0].cpu().numpy(), ref + (sb ** 2).sum(1)) <= NORM_GATE["f32"]
