"""GPU parity of gws_linear_bwd_w: the weight-gradient GEMM dW = X^T dY with the block reduction of the
paper's Eq. 4 in its epilogue.  dW is checked against the fp64 oracle GEMM (one BF16 rounding + fp32
accumulation in any order); dL/db_t is checked against the oracle's backward pass on the very dW bytes
the GPU produced (the reduction is defined on the rounded BF16 gradient), to the 1e-5 bar."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_11170_amd as gws
from paper_2505_11170_amd import synth
from gpu_util import DEV, assert_dbt_close, ensure_built

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


def f64(bits):
    return (np.ascontiguousarray(bits).astype(np.uint32) << 16).view(np.float32).astype(np.float64)


def run_case(M, K, N, w_is_nk, idx, step=4, rows_sel=None, pad=0, row0=0, col0=0, split=None):
    """split: None = gws_linear_bwd_w; a number of bytes = gws_linear_bwd_w_ws with a workspace of that size
    (-1: the size gws_linear_bwd_w_workspace_bytes names, which must then be positive)."""
    x = synth.make_activation(idx, M, K)
    dy = (synth.make_activation(idx + 1, M, N).float() * 1e-3).to(torch.bfloat16)   # upstream gradient ~ N(0, 1e-3)
    rows, cols = (N, K) if w_is_nk else (K, N)
    ld = cols + pad
    nbr, nbc = rows // 32, cols // 32
    gen = torch.Generator().manual_seed(9000 + idx)
    scale = (torch.rand(nbr, nbc, generator=gen) * 1e-3 + 1e-5).float()
    seed = oracle.derive_seed(2, idx)
    dw = torch.zeros(rows, ld, dtype=torch.bfloat16, device=DEV)
    dbt = torch.full((nbr, nbc), float("nan"), device=DEV)
    d = gws.TensorDesc(rows=rows, cols=cols, seed=seed, scale=scale.to(DEV), dw=dw, dbt=dbt, ld=ld, row0=row0, col0=col0)
    xg, dyg = x.to(DEV), dy.to(DEV)
    if split is None:
        gws.gws_linear_bwd_w(xg, dyg, d, step, w_is_nk=w_is_nk)
    else:
        want = gws.gws_linear_bwd_w_workspace_bytes(d, M)
        if split < 0:
            assert want > 0, ("no split planned", M, K, N)
            split = want
        ws = torch.full((max(split, 16) // 4,), float("nan"), device=DEV)          # stale contents must not matter
        gws.gws_linear_bwd_w_ws(xg, dyg, d, step, ws[: split // 4], w_is_nk=w_is_nk)
    torch.cuda.synchronize()
    dw_bits = synth.bits(dw)
    assert (dw_bits[:, cols:] == 0).all()                       # padding columns are never written
    # dW against the fp64 GEMM: rows of dW are columns of A (X, or dY for the [N x K] layout)
    a, b = (dy, x) if w_is_nk else (x, dy)
    at = np.ascontiguousarray(synth.bits(a).T)
    sel = None if rows_sel is None else np.asarray(rows_sel)
    y64, yabs, _ = oracle.linear_fwd(at, synth.bits(b), rows_sel=sel)
    got = f64(dw_bits[:, :cols] if sel is None else dw_bits[sel, :cols])
    tol = 2.0 ** -8 * np.abs(y64) + M * 2.0 ** -24 * yabs + 1e-30
    assert (np.abs(got - y64) <= tol).all(), ("dW", M, K, N, w_is_nk)
    # dL/db_t against the oracle's Eq. 4 on the GPU's own dW bytes
    _, ref_dbt, asum = oracle.sample_bwd(np.ascontiguousarray(dw_bits), scale.numpy(), seed, step, cols=cols, row0=row0, col0=col0)
    assert_dbt_close(dbt.cpu().numpy(), ref_dbt, asum, ("dbt", M, K, N, w_is_nk))
    return xg, dyg, d, dw_bits, dbt.cpu().numpy()


@pytest.mark.parametrize("w_is_nk", [False, True])
def test_single_tile_and_several_tiles(w_is_nk):
    # few tiles of 256 x 256: small pieces (the other forms: test_each_form_padded_sharded_and_without_the_reduction)
    run_case(64, 256, 256, w_is_nk, 800)
    run_case(192, 512, 768, w_is_nk, 802, pad=8)
    run_case(128, 768, 256, w_is_nk, 804, row0=256, col0=512)     # a shard: the origin enters the noise counter


def test_every_number_of_k_steps():
    # tokens are the contraction here: 1 .. 13 units of 64 tokens for the four wavefronts of a small piece (the tiles' own
    # loops: test_every_form_of_the_weight_gradient)
    for nk in range(1, 14):
        run_case(64 * nk, 256, 256, bool(nk & 1), 840 + 2 * nk)


@pytest.mark.parametrize("w_is_nk", [False, True])
def test_config5_shape(w_is_nk):
    M, K, N = 8192, 2048, 5632
    rows = N if w_is_nk else K
    # one row of dW in every 256-row tile of the weight, at a different 32-row sub-tile each time, plus the ends
    rng = np.random.default_rng(810)
    sel = sorted({0, rows - 1} | {t * 256 + 32 * (t % 8) + int(rng.integers(0, 32)) for t in range(rows // 256)})
    run_case(M, K, N, w_is_nk, 810, rows_sel=sel)


def test_epilogue_agrees_with_the_separate_backward_kernel_and_plain_form():
    xg, dyg, d, dw_bits, dbt = run_case(256, 512, 512, False, 820)
    # the same dW without the reduction
    dw2 = torch.zeros_like(d.dw)
    d2 = gws.TensorDesc(rows=d.rows, cols=d.cols, seed=d.seed, dw=dw2, ld=d.ld)
    gws.gws_linear_bwd_w(xg, dyg, d2, 4)
    # and the separate kernel on those bytes
    dbt3 = torch.zeros_like(d.dbt)
    d3 = gws.TensorDesc(rows=d.rows, cols=d.cols, seed=d.seed, g=d.dw, dw=d.dw, dbt=dbt3, scale=d.scale, ld=d.ld)
    gws.gws_sample_bwd([d3], 4)
    torch.cuda.synchronize()
    assert (synth.bits(dw2) == dw_bits).all()
    a, b = dbt3.cpu().numpy().astype(np.float64), dbt.astype(np.float64)
    _, _, asum = oracle.sample_bwd(np.ascontiguousarray(dw_bits), d.scale.cpu().numpy(), d.seed, 4)
    assert (np.abs(a - b) <= 1e-5 * np.abs(a) + 2e-6 * asum).all()


@pytest.mark.parametrize("w_is_nk", [False, True])
def test_tokens_split_into_parts(w_is_nk):
    # few tokens: small pieces of the gradient, with as many sums as the workspace holds parts or more
    run_case(1024, 256, 256, w_is_nk, 860, split=-1)                  # 1 tile, room for 2 parts: four sums
    run_case(2048, 512, 768, w_is_nk, 862, pad=8, split=-1)           # 6 tiles, room for 4 parts: four sums
    run_case(4352, 768, 256, w_is_nk, 864, row0=256, col0=512, split=-1)   # 3 tiles, room for 8 parts: eight sums of 8 or 9 units
    # a workspace with room for three parts where eight were planned, and none at all
    per_part = 3 * 256 * 256 * 4
    run_case(4352, 768, 256, w_is_nk, 866, split=3 * per_part + 100)
    run_case(1024, 256, 256, w_is_nk, 868, split=0)
    # many tokens: the contraction is split (partial tiles go through the workspace and are added in a fixed order), uneven
    # where the units do not divide; dW and dL/db_t to the same bars
    for tokens, K, N, idx in [(8192, 512, 512, 870), (5184, 256, 256, 872)]:
        assert gws.gws_linear_bwd_w_form(gws.TensorDesc(rows=K, cols=N, ld=N, seed=0), tokens, 8 * K * N * 4, on_lines=False) == gws.BWD_W_SPLIT + 8
        run_case(tokens, K, N, w_is_nk, idx, pad=8, row0=256, col0=512, split=-1)


def test_config5_sized_weights_split_over_tokens():
    # the 2048 x 2048 weight of the 1B layer over 8192 tokens: in pieces of 128 x 128, and with rows off the cache lines
    # 64 tiles in 4 parts; a row in every 256-row tile
    rng = np.random.default_rng(870)
    sel = sorted({0, 2047} | {t * 256 + int(rng.integers(0, 256)) for t in range(8)})
    d = gws.TensorDesc(rows=2048, cols=2048, ld=2048, seed=0)
    assert gws.gws_linear_bwd_w_form(d, 8192, 1 << 30) == gws.BWD_W_PIECES_128_128
    run_case(8192, 2048, 2048, False, 870, rows_sel=sel, split=-1)
    assert gws.gws_linear_bwd_w_form(d, 8192, 1 << 30, on_lines=False) == gws.BWD_W_SPLIT + 4
    run_case(8192, 2048, 2048, False, 871, pad=8, rows_sel=sel, split=-1)
    d = gws.TensorDesc(rows=2048, cols=5632, seed=1)
    assert gws.gws_linear_bwd_w_workspace_bytes(d, 8192) == 0          # 176 tiles: the one-kernel form
    assert gws.gws_linear_bwd_w_workspace_bytes(gws.TensorDesc(rows=2048, cols=2048, seed=1), 8192) == 4 * 64 * 256 * 256 * 4


def test_workspace_argument_errors():
    x = torch.zeros(1024, 256, dtype=torch.bfloat16, device=DEV)
    dy = torch.zeros(1024, 256, dtype=torch.bfloat16, device=DEV)
    dw = torch.zeros(256, 256, dtype=torch.bfloat16, device=DEV)
    d = gws.TensorDesc(rows=256, cols=256, seed=1, dw=dw)
    need = gws.gws_linear_bwd_w_workspace_bytes(d, 1024)
    assert need == 2 * 256 * 256 * 4
    ws = torch.zeros(need // 4 + 4, device=DEV)
    with pytest.raises(gws.GwsError) as e:
        gws.gws_linear_bwd_w_ws(x, dy, d, 0, ws.view(torch.uint8)[4: 4 + need])      # not 16-byte aligned
    assert e.value.status == 3
    with pytest.raises(gws.GwsError) as e:
        gws.gws_linear_bwd_w_ws(x, dy, gws.TensorDesc(rows=256, cols=256, seed=1, dw=ws.view(torch.bfloat16)[:65536].view(256, 256)), 0, ws)
    assert e.value.status == 6                                                          # workspace on top of dW
    torch.cuda.synchronize()


def test_shape_and_argument_errors():
    x = torch.zeros(64, 256, dtype=torch.bfloat16, device=DEV)
    dy = torch.zeros(64, 256, dtype=torch.bfloat16, device=DEV)
    dw = torch.zeros(256, 256, dtype=torch.bfloat16, device=DEV)
    sc = torch.ones(8, 8, device=DEV)
    ok = gws.TensorDesc(rows=256, cols=256, seed=1, dw=dw, dbt=torch.zeros(8, 8, device=DEV), scale=sc)
    gws.gws_linear_bwd_w(x, dy, ok, 0)
    for bad, status in [(gws.TensorDesc(rows=128, cols=256, seed=1, dw=dw), 2),            # rows not a multiple of 256
                        (gws.TensorDesc(rows=256, cols=256, seed=1, dw=None), 1),
                        (gws.TensorDesc(rows=256, cols=256, seed=1, dw=dw, dbt=sc), 1)]:   # dbt without scale
        with pytest.raises(gws.GwsError) as e:
            gws.gws_linear_bwd_w(x, dy, bad, 0)
        assert e.value.status == status
    with pytest.raises(gws.GwsError) as e:
        gws.gws_linear_bwd_w(x[:32], dy[:32], ok, 0)                                       # M not a multiple of 64
    assert e.value.status == 2
    with pytest.raises(gws.GwsError) as e:
        gws.gws_linear_bwd_w(x, dy, gws.TensorDesc(rows=256, cols=256, seed=1, dw=x), 0)   # dW on top of X
    assert e.value.status == 6
    torch.cuda.synchronize()


def test_random_shapes():
    # seeded random weight shapes (multiples of 256) and token counts (multiples of 64: 1 .. 9 K-steps)
    rng = np.random.default_rng(1117)
    for case in range(6):
        K, N = 256 * int(rng.integers(1, 4)), 256 * int(rng.integers(1, 4))
        M = 64 * int(rng.integers(1, 10))
        run_case(M, K, N, bool(case & 1), 830 + 2 * case, pad=8 * int(rng.integers(0, 3)))


def fp32_product(a, b):
    """a^T b in fp32 on the GPU (a, b [tokens x n])."""
    return a.float().t().contiguous() @ b.float()


@pytest.mark.parametrize("tokens,rows,cols", [(64 * i, 4096, 4096) for i in range(1, 15)] + [(64 * i, 2048, 5632) for i in range(6, 20)] + [(8192, 2048, 2048), (4096, 768, 3072), (8192, 512, 512)]
                         + [(64, 256, 256), (128, 256, 512), (320, 512, 768), (576, 1536, 1024), (1600, 1280, 1024)])
def test_every_form_of_the_weight_gradient(tokens, rows, cols):
    # one workgroup per 256 x 256 or 256 x 192 tile (256 and 240 tiles, every number of K-steps around the rings' period), the tokens split over
    # workgroups (all the workspace, room for two parts), small pieces with the tokens split over wavefronts (fewer units of
    # 64 tokens than wavefronts, uneven numbers of them): dW to its rounding and the order of fp32 sums, and dL/db_t to the
    # separate kernel's on the same bytes
    gen = torch.Generator(device=DEV).manual_seed(tokens + rows)
    x = torch.randn(tokens, rows, generator=gen, device=DEV).to(torch.bfloat16)
    dy = (torch.randn(tokens, cols, generator=gen, device=DEV) * 1e-3).to(torch.bfloat16)
    d = gws.TensorDesc(rows=rows, cols=cols, seed=77, scale=torch.rand(rows // 32, cols // 32, generator=gen, device=DEV),
                       dw=torch.zeros(rows, cols, dtype=torch.bfloat16, device=DEV), dbt=torch.zeros(rows // 32, cols // 32, device=DEV))
    ref, mag = fp32_product(x, dy), fp32_product(x.abs(), dy.abs())
    need = gws.gws_linear_bwd_w_workspace_bytes(d, tokens)
    for nbytes in {0, need, min(need, 2 * rows * cols * 4)}:
        d.dw.zero_()
        d.dbt.zero_()
        gws.gws_linear_bwd_w_ws(x, dy, d, 5, torch.empty(nbytes, dtype=torch.uint8, device=DEV) if nbytes else None)
        # one rounding to BF16 and two fp32 sums of `tokens` terms in different orders
        assert bool(((d.dw.float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2 * tokens * 2.0 ** -24 * mag).all()), nbytes
        back = gws.TensorDesc(rows=rows, cols=cols, seed=77, scale=d.scale, g=d.dw, dw=None, dbt=torch.zeros_like(d.dbt), ld=cols)
        gws.gws_sample_bwd([back], 5)
        terms = 0.6932 * d.scale * d.dw.float().abs().view(rows // 32, 32, cols // 32, 32).sum((1, 3)) * 2
        assert bool(((d.dbt - back.dbt).abs() <= 1e-5 * back.dbt.abs() + 1e-6 * terms).all()), nbytes


@pytest.mark.parametrize("tokens,rows,cols", [(4096, 768, 3072), (1024, 2048, 4096), (8192, 1024, 1024), (8192, 512, 512), (1536, 1536, 1024), (8192, 2048, 2048)])
def test_no_fp32_sum_runs_over_more_tokens_than_a_part_of_the_workspace(tokens, rows, cols):
    # Every element of dW is 2^27 (first token) + ones - 2^27 (last token).  In fp32 the 2^27 (spacing 16) swallows the
    # ones that the same sum meets after it, at most eight of 32 tokens at once; 16 of 64 tokens are ones, so sums that
    # have not met it add to it exactly.  The ones that are missing say over how many tokens the first sum ran.
    units = tokens // 64
    one = (torch.arange(tokens) % 4 == 1) & (torch.arange(tokens) >= 32) & (torch.arange(tokens) < tokens - 32)
    x = torch.zeros(tokens, rows, dtype=torch.bfloat16)
    dy = torch.zeros(tokens, cols, dtype=torch.bfloat16)
    x[one], dy[one] = 1.0, 1.0
    x[0], x[-1], dy[0], dy[-1] = 2.0 ** 14, 2.0 ** 14, 2.0 ** 13, -2.0 ** 13
    d = gws.TensorDesc(rows=rows, cols=cols, seed=3, dw=torch.zeros(rows, cols, dtype=torch.bfloat16, device=DEV))
    part_bytes = rows * cols * 4
    need = gws.gws_linear_bwd_w_workspace_bytes(d, tokens)
    assert need >= 2 * part_bytes
    for parts in sorted({2, need // part_bytes}):
        gws.gws_linear_bwd_w_ws(x.to(DEV), dy.to(DEV), d, 5, torch.empty(parts * part_bytes, dtype=torch.uint8, device=DEV))
        got = d.dw.float()
        total, run = int(one.sum()), -(-units // parts)
        assert float(got.max()) <= total
        lost = total - float(got.min())
        assert lost <= 16 * run + 2.0 ** -8 * total, (parts, lost / 16, run)   # what the rounding to BF16 may add


PIECES, SPLIT = {gws.BWD_W_PIECES_32, gws.BWD_W_PIECES_64, gws.BWD_W_PIECES_96, gws.BWD_W_PIECES_128, gws.BWD_W_PIECES_128_128}, gws.BWD_W_SPLIT


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("form,tokens,rows,cols,room", [
    ({gws.BWD_W_WIDE}, 64, 4096, 4096, 0), ({gws.BWD_W_WIDE}, 448, 4096, 4096, 0), ({gws.BWD_W_WIDE}, 192, 2048, 5632, 0), ({gws.BWD_W_NARROW}, 832, 2048, 5632, 0), ({gws.BWD_W_NARROW}, 1088, 2048, 5632, 0),
    (PIECES, 192, 512, 768, 0), (PIECES, 576, 1536, 1024, 0), (PIECES, 2048, 1024, 1024, 4), (PIECES, 4096, 768, 768, 8), (PIECES, 4096, 768, 2304, 8),
    ({SPLIT + 2}, 3584, 2048, 2816, 2), (PIECES, 4096, 768, 3072, 2), ({SPLIT + 3}, 2560, 1536, 2816, 3), ({SPLIT + 5}, 2560, 1280, 1792, 5), ({SPLIT + 6}, 3072, 1280, 1792, 6), ({SPLIT + 7}, 3584, 1280, 1792, 7), (PIECES, 1088, 2048, 4096, 2),
    ({SPLIT + 8}, 6656, 512, 2304, 8), ({SPLIT + 8}, 8192, 512, 512, 8)])
def test_each_form_padded_sharded_and_without_the_reduction(form, tokens, rows, cols, room, w_is_nk):
    # X and dY in wider buffers with NaN beside them, dW in a wider buffer, the weight a shard of a larger one; room: the
    # parts that the workspace holds.  With dL/db_t and without, the same dW
    gen = torch.Generator(device=DEV).manual_seed(tokens + rows)
    K, N = (cols, rows) if w_is_nk else (rows, cols)
    x = torch.full((tokens, K + 24), float("nan"), dtype=torch.bfloat16, device=DEV)
    dy = torch.full((tokens, N + 8), float("nan"), dtype=torch.bfloat16, device=DEV)
    x[:, :K] = torch.randn(tokens, K, generator=gen, device=DEV)
    dy[:, :N] = torch.randn(tokens, N, generator=gen, device=DEV) * 1e-3
    dw = torch.full((rows, cols + 16), 7.0, dtype=torch.bfloat16, device=DEV)
    shard = dict(rows=rows, cols=cols, ld=cols + 16, row0=320, col0=96, seed=41)
    d = gws.TensorDesc(**shard, dw=dw, scale=torch.rand(rows // 32, cols // 32, generator=gen, device=DEV), dbt=torch.full((rows // 32, cols // 32), float("nan"), device=DEV))
    ws = torch.full((room * rows * cols,), float("nan"), device=DEV) if room else None
    assert gws.gws_linear_bwd_w_form(d, tokens, room * rows * cols * 4, on_lines=False) in form
    gws.gws_linear_bwd_w_ws(x[:, :K], dy[:, :N], d, 5, ws, w_is_nk=w_is_nk)
    a, b = (dy[:, :N], x[:, :K]) if w_is_nk else (x[:, :K], dy[:, :N])
    ref, mag = fp32_product(a, b), fp32_product(a.abs(), b.abs())
    # one rounding to BF16 and two fp32 sums of `tokens` terms in different orders
    assert bool(((dw[:, :cols].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2 * tokens * 2.0 ** -24 * mag).all())
    assert bool((dw[:, cols:] == 7.0).all())
    back = gws.TensorDesc(**shard, scale=d.scale, g=dw, dw=None, dbt=torch.zeros_like(d.dbt))
    gws.gws_sample_bwd([back], 5)
    terms = 0.6932 * d.scale * dw[:, :cols].float().abs().view(rows // 32, 32, cols // 32, 32).sum((1, 3)) * 2
    assert bool(((d.dbt - back.dbt).abs() <= 1e-5 * back.dbt.abs() + 1e-6 * terms).all())
    with_dbt = dw.clone()
    dw.fill_(7.0)
    gws.gws_linear_bwd_w_ws(x[:, :K], dy[:, :N], gws.TensorDesc(**shard, dw=dw), 5, ws, w_is_nk=w_is_nk)
    assert torch.equal(dw.view(torch.int16), with_dbt.view(torch.int16))


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("form,tokens,rows,cols,room", [
    (gws.BWD_W_PIECES_32, 64, 256, 256, 0), (gws.BWD_W_PIECES_32, 448, 256, 512, 0), (gws.BWD_W_PIECES_32, 8192, 256, 2048, 8),
    (gws.BWD_W_PIECES_96, 64, 768, 2816, 0), (gws.BWD_W_PIECES_96, 448, 1280, 3328, 0), (gws.BWD_W_PIECES_96, 2624, 768, 2816, 5), (gws.BWD_W_PIECES_96, 4096, 768, 3072, 7),
    (gws.BWD_W_PIECES_128_128, 64, 1280, 1792, 0), (gws.BWD_W_PIECES_128_128, 832, 2048, 2048, 0), (gws.BWD_W_PIECES_128_128, 1088, 2048, 4096, 2),
    (gws.BWD_W_PIECES_32, 448, 512, 256, 0), (gws.BWD_W_PIECES_32, 2240, 1792, 256, 0), (gws.BWD_W_PIECES_96, 64, 2816, 768, 0), (gws.BWD_W_PIECES_96, 448, 3328, 1280, 0),
    (gws.BWD_W_PIECES_128_128, 832, 2304, 1792, 0), (gws.BWD_W_PIECES_128, 1344, 3072, 512, 0), (gws.BWD_W_PIECES_64, 4096, 1280, 512, 0)])
def test_pieces_for_rows_on_cache_lines(form, tokens, rows, cols, room, w_is_nk):
    # weights wider and taller than square (the pieces are dealt along the longer side), fewer units of tokens than wavefronts, uneven numbers of them, pieces past the weight's edge, sums in two halves; X and
    # dY in wider buffers with NaN beside them, the weight a shard of a larger one, dW in a wider buffer
    gen = torch.Generator(device=DEV).manual_seed(tokens + cols)
    K, N = (cols, rows) if w_is_nk else (rows, cols)
    x = torch.full((tokens, K + 64), float("nan"), dtype=torch.bfloat16, device=DEV)
    dy = torch.full((tokens, N + 64), float("nan"), dtype=torch.bfloat16, device=DEV)
    x[:, :K] = torch.randn(tokens, K, generator=gen, device=DEV)
    dy[:, :N] = torch.randn(tokens, N, generator=gen, device=DEV) * 1e-3
    dw = torch.full((rows, cols + 64), 7.0, dtype=torch.bfloat16, device=DEV)
    shard = dict(rows=rows, cols=cols, ld=cols + 64, row0=320, col0=96, seed=41)
    d = gws.TensorDesc(**shard, dw=dw, scale=torch.rand(rows // 32, cols // 32, generator=gen, device=DEV), dbt=torch.full((rows // 32, cols // 32), float("nan"), device=DEV))
    ws = torch.full((room * rows * cols,), float("nan"), device=DEV) if room else None
    assert gws.gws_linear_bwd_w_form(d, tokens, room * rows * cols * 4, on_lines=True) == form
    gws.gws_linear_bwd_w_ws(x[:, :K], dy[:, :N], d, 5, ws, w_is_nk=w_is_nk)
    a, b = (dy[:, :N], x[:, :K]) if w_is_nk else (x[:, :K], dy[:, :N])
    ref, mag = fp32_product(a, b), fp32_product(a.abs(), b.abs())
    # one rounding to BF16 and two fp32 sums of `tokens` terms in different orders
    assert bool(((dw[:, :cols].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2 * tokens * 2.0 ** -24 * mag).all())
    assert bool((dw[:, cols:] == 7.0).all())
    back = gws.TensorDesc(**shard, scale=d.scale, g=dw, dw=None, dbt=torch.zeros_like(d.dbt))
    gws.gws_sample_bwd([back], 5)
    terms = 0.6932 * d.scale * dw[:, :cols].float().abs().view(rows // 32, 32, cols // 32, 32).sum((1, 3)) * 2
    assert bool(((d.dbt - back.dbt).abs() <= 1e-5 * back.dbt.abs() + 1e-6 * terms).all())
    with_dbt = dw.clone()
    dw.fill_(7.0)
    gws.gws_linear_bwd_w_ws(x[:, :K], dy[:, :N], gws.TensorDesc(**shard, dw=dw), 5, ws, w_is_nk=w_is_nk)
    assert torch.equal(dw.view(torch.int16), with_dbt.view(torch.int16))


# pieces by 2 x 2 wavefronts: fewer stages of 64 tokens than the ring holds, as many, one more, and the last token counts before and the
# first after which a piece's tokens are split over the wavefronts, multiples of 256 and others; room: a workspace of so many parts, of which the tokens make one to
# three (the kernel has four fp32 sums whatever the workspace holds)
@pytest.mark.parametrize("form,tokens,rows,cols,room", [
    (gws.BWD_W_PIECES_32, 128, 256, 512, 0), (gws.BWD_W_PIECES_32, 192, 256, 512, 0), (gws.BWD_W_PIECES_64, 64, 768, 768, 0), (gws.BWD_W_PIECES_64, 128, 1024, 768, 8),
    (gws.BWD_W_PIECES_64, 192, 768, 768, 0), (gws.BWD_W_PIECES_128, 320, 1280, 1024, 0), (gws.BWD_W_PIECES_128, 384, 768, 2304, 8), (gws.BWD_W_PIECES_128, 448, 512, 3328, 0),
    (gws.BWD_W_PIECES_128, 1216, 768, 2304, 8), (gws.BWD_W_PIECES_128, 1280, 768, 2304, 0), (gws.BWD_W_PIECES_96, 384, 768, 2816, 8), (gws.BWD_W_PIECES_96, 1408, 2816, 768, 0),
    (gws.BWD_W_PIECES_96, 1472, 768, 2816, 0), (gws.BWD_W_PIECES_128_128, 256, 2048, 1792, 0), (gws.BWD_W_PIECES_128_128, 320, 1280, 1792, 0),
    (gws.BWD_W_PIECES_128_128, 384, 1024, 3328, 8), (gws.BWD_W_PIECES_128_128, 1664, 1536, 2048, 8), (gws.BWD_W_PIECES_96, 960, 768, 2816, 8),
    (gws.BWD_W_PIECES_96, 1024, 2816, 768, 0), (gws.BWD_W_PIECES_128_128, 2048, 1024, 2304, 8), (gws.BWD_W_PIECES_128_128, 2304, 1280, 1792, 0),
    (gws.BWD_W_PIECES_128_128, 2240, 1024, 2304, 8), (gws.BWD_W_PIECES_128_128, 4160, 1280, 1792, 0)])
def test_pieces_by_wavefronts_that_walk_the_tokens_together(form, tokens, rows, cols, room):
    nk = bool(tokens & 64)
    d = gws.TensorDesc(rows=rows, cols=cols, seed=1, dw=torch.empty(rows, cols, dtype=torch.bfloat16, device=DEV))
    size = min(room, 8) * rows * cols * 4
    assert gws.gws_linear_bwd_w_form(d, tokens, size) == form
    K, N = (cols, rows) if nk else (rows, cols)
    sel = range(0, rows, 61) if rows * cols * tokens > 1 << 30 else None
    run_case(tokens, K, N, nk, 960 + tokens // 64, rows_sel=sel, split=size if size else None)
