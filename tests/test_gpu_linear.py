"""GPU parity of gws_linear_fwd / gws_linear_fwd_mode / gws_linear_fwd_ws (the sampled-weight
linear in its forms: sampling in the weight operand load, sampling kernel + plain GEMM with w_hat
in the caller's buffer or staged in a workspace) and of the plain twin gws_gemm_bf16, through the C ABI.

 - w_hat / scale written by the call: bit-exact against the oracle forward.
 - Y against the oracle's fp64 GEMM on the oracle's w_hat: |y - ref| <= 2^-8 |ref| +
   K * 2^-24 * sum|x q| (one BF16 rounding plus fp32 accumulation in any order).
 - fused Y == plain GEMM on the separately sampled w_hat, bit for bit (same GEMM code).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_11170_amd as gws
from paper_2505_11170_amd import synth
from gpu_util import DEV, ensure_built

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


def bf16_val(bits):
    return (np.ascontiguousarray(bits, dtype=np.uint16).astype(np.uint32) << 16).view(np.float32).astype(np.float64)


def check_y(y_bits, x_bits, q_bits, w_is_nk, rows_sel=None):
    K = x_bits.shape[1]
    y64, yabs, _ = oracle.linear_fwd(x_bits, q_bits, w_is_nk=w_is_nk, rows_sel=rows_sel)
    got = bf16_val(y_bits if rows_sel is None else y_bits[rows_sel])
    tol = 2.0 ** -8 * np.abs(y64) + K * 2.0 ** -24 * yabs + 1e-30
    bad = np.abs(got - y64) > tol
    assert not bad.any(), (np.argwhere(bad)[:5], got[bad][:5], y64[bad][:5])


def run_case(M, K, N, w_is_nk, fmt, bt=None, seed_id=0, step=0, rows_sel=None, ldx_pad=0, ldy_pad=0, mode=None):
    wr, wc = (N, K) if w_is_nk else (K, N)
    t = synth.make_tensor(200 + seed_id, wr, wc, bt=bt, with_grad=False)
    x_full = synth.make_activation(300 + seed_id, M, K + ldx_pad)
    x = x_full.to(DEV)[:, :K]
    w = t["w"].to(DEV)
    btd = t["bt"].to(DEV)
    seed = oracle.derive_seed(0, seed_id)
    y_store = torch.zeros(M, N + ldy_pad, dtype=torch.bfloat16, device=DEV)
    y = y_store[:, :N]
    w_hat = torch.zeros_like(w)
    nbr, nbc = synth.n_blocks(wr, wc)
    scale = torch.zeros(nbr, nbc, dtype=torch.float32, device=DEV)
    desc = gws.TensorDesc(rows=wr, cols=wc, seed=seed, w=w, w_hat=w_hat, bt=btd, scale=scale)
    if mode is None:
        gws.gws_linear_fwd(x, desc, y, fmt, step, w_is_nk=w_is_nk)
    else:
        gws.gws_linear_fwd_mode(x, desc, y, fmt, step, mode, w_is_nk=w_is_nk)
    torch.cuda.synchronize()
    # 1. sampled weight written by the call == oracle
    ref_q, ref_s = oracle.sample_fwd(synth.bits(t["w"]), t["bt"].numpy(), fmt, seed, step)
    assert (synth.bits(w_hat) == ref_q).all()
    assert (scale.cpu().numpy().view(np.uint32) == ref_s.view(np.uint32)).all()
    # 2. Y against the fp64 GEMM
    x_bits = np.ascontiguousarray(synth.bits(x_full)[:, :K])
    y_bits = np.ascontiguousarray(synth.bits(y_store)[:, :N])
    check_y(y_bits, x_bits, ref_q, w_is_nk, rows_sel)
    if ldy_pad:
        assert (synth.bits(y_store)[:, N:] == 0).all()          # padding of Y never written
    # 3. unfused path (sample kernel + plain GEMM) gives the same bits
    w_hat2 = torch.zeros_like(w)
    scale2 = torch.zeros_like(scale)
    gws.gws_sample_fwd([gws.TensorDesc(rows=wr, cols=wc, seed=seed, w=w, w_hat=w_hat2, bt=btd, scale=scale2)], fmt, step)
    y2 = torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)
    gws.gws_gemm_bf16(x, w_hat2, y2, w_is_nk=w_is_nk)
    torch.cuda.synchronize()
    assert (synth.bits(w_hat2) == ref_q).all()
    assert (synth.bits(y2) == y_bits).all()
    # 4. without w_hat / scale outputs the result is the same
    y3 = torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)
    gws.gws_linear_fwd(x, gws.TensorDesc(rows=wr, cols=wc, seed=seed, w=w, bt=btd), y3, fmt, step, w_is_nk=w_is_nk)
    torch.cuda.synchronize()
    assert (synth.bits(y3) == y_bits).all()
    # 5. ... and with w_hat staged in a caller's workspace (poisoned first, oversized: the tail stays as it was)
    bare = gws.TensorDesc(rows=wr, cols=wc, seed=seed, w=w, bt=btd)
    need = gws.gws_linear_fwd_workspace_bytes(bare)
    assert need == ((wr * wc * 2 + 255) // 256) * 256 + 4 * nbr * nbc
    ws = torch.full((need + 512,), 0xA5, dtype=torch.uint8, device=DEV)
    y4 = torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)
    gws.gws_linear_fwd_ws(x, bare, y4, fmt, step, ws, w_is_nk=w_is_nk)
    torch.cuda.synchronize()
    assert (synth.bits(y4) == y_bits).all()
    assert (ws[need:] == 0xA5).all()


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("fmt", [gws.FMT_BF16, gws.FMT_FP8_E4M3, gws.FMT_FP6_E3M2])
def test_linear_small_shapes(w_is_nk, fmt):
    run_case(128, 64, 128, w_is_nk, fmt, bt=6.0)                    # automatic choice (w_hat given: sampling kernel + GEMM)
    run_case(200, 96, 160, w_is_nk, fmt, seed_id=1)                 # two kernels; ragged M, N not a tile multiple
    run_case(37, 32, 32, w_is_nk, fmt, seed_id=2, step=3)
    run_case(300, 256, 416, w_is_nk, fmt, seed_id=3, ldx_pad=8, ldy_pad=16)
    run_case(200, 96, 160, w_is_nk, fmt, seed_id=1, mode=gws.LINEAR_IN_OPERAND)
    run_case(300, 256, 416, w_is_nk, fmt, seed_id=3, ldx_pad=8, ldy_pad=16, mode=gws.LINEAR_IN_OPERAND)
    run_case(37, 32, 32, w_is_nk, fmt, seed_id=2, step=3, mode=gws.LINEAR_TWO_KERNELS)


def test_plain_gemm_vs_fp64():
    M, K, N = 260, 192, 224
    x = synth.make_activation(1, M, K)
    w = synth.make_tensor(1, K, N, with_grad=False)["w"]
    y = torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)
    gws.gws_gemm_bf16(x.to(DEV), w.to(DEV), y)
    torch.cuda.synchronize()
    check_y(synth.bits(y), synth.bits(x), synth.bits(w), False)
    wt = w.t().contiguous()
    y2 = torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)
    gws.gws_gemm_bf16(x.to(DEV), wt.to(DEV), y2, w_is_nk=True)
    torch.cuda.synchronize()
    check_y(synth.bits(y2), synth.bits(x), synth.bits(wt), True)


@pytest.mark.parametrize("w_is_nk", [False, True])
def test_plain_gemm_large_tile_path(w_is_nk):
    # whole 256 x 256 tiles but few of them: the kernel that splits K (the large tile itself: 10 x 19 tiles below, which
    # exercise the XCD / patch tile numbering with a short last band)
    large = (2560, 64, 4864)
    assert gws.gws_gemm_form(*large, w_is_nk) == gws.GEMM_LARGE
    x = synth.make_activation(9, large[0], large[1])
    w = synth.make_tensor(9, large[1], large[2], with_grad=False)["w"]
    wd = (w.t().contiguous() if w_is_nk else w).to(DEV)
    y = torch.zeros(large[0], large[2], dtype=torch.bfloat16, device=DEV)
    gws.gws_gemm_bf16(x.to(DEV), wd, y, w_is_nk=w_is_nk)
    torch.cuda.synchronize()
    check_y(synth.bits(y), synth.bits(x), synth.bits(wd.cpu()), w_is_nk, tile_rows(large[0], np.random.default_rng(9)))
    M, K, N = 768, 192, 1280
    x = synth.make_activation(2, M, K)
    w = synth.make_tensor(2, K, N, with_grad=False)["w"]
    wd = (w.t().contiguous() if w_is_nk else w).to(DEV)
    y = torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)
    gws.gws_gemm_bf16(x.to(DEV), wd, y, w_is_nk=w_is_nk)
    torch.cuda.synchronize()
    check_y(synth.bits(y), synth.bits(x), synth.bits(wd.cpu()), w_is_nk)
    # a 9 x 2 tile grid: more than one band of 8 m-tiles
    M2, K2, N2 = 2304, 64, 512
    x2 = synth.make_activation(3, M2, K2)
    w2 = synth.make_tensor(3, K2, N2, with_grad=False)["w"]
    wd2 = (w2.t().contiguous() if w_is_nk else w2).to(DEV)
    y2 = torch.zeros(M2, N2, dtype=torch.bfloat16, device=DEV)
    gws.gws_gemm_bf16(x2.to(DEV), wd2, y2, w_is_nk=w_is_nk)
    torch.cuda.synchronize()
    check_y(synth.bits(y2), synth.bits(x2), synth.bits(wd2.cpu()), w_is_nk)


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("fmt", [gws.FMT_BF16, gws.FMT_FP8_E4M3, gws.FMT_FP6_E3M2])
def test_linear_on_the_large_tile(w_is_nk, fmt):
    # w_hat requested: sampling kernel + the 256-tile GEMM on w_hat; with few tiles the GEMM that splits K
    assert gws.gws_gemm_form(2560, 64, 4864, w_is_nk, sampled=2) == gws.GEMM_LARGE
    run_case(2560, 64, 4864, w_is_nk, fmt, seed_id=10, step=3, rows_sel=tile_rows(2560, np.random.default_rng(10)))
    run_case(512, 128, 768, w_is_nk, fmt, seed_id=7, step=2)
    run_case(256, 64, 256, w_is_nk, fmt, bt=3.0, seed_id=8)


def tile_rows(M, rng, tile=256, sub=32):
    """One row in every `tile`-row output tile, at a different 32-row MFMA sub-tile and lane row each time,
    plus the first and last row: every M-tile and, over the tiles, every wavefront quadrant is hit."""
    rows = {0, M - 1}
    for t in range(M // tile):
        rows.add(t * tile + sub * (t % (tile // sub)) + int(rng.integers(0, sub)))
    return np.array(sorted(rows))


def test_config5_fused_linear_8192x2048x5632_a_row_in_every_tile():
    M, K, N = 8192, 2048, 5632
    rows_sel = tile_rows(M, np.random.default_rng(5))
    assert len(rows_sel) >= 32 and len(set(rows_sel // 256)) == 32
    for mode in (None, gws.LINEAR_IN_OPERAND):
        run_case(M, K, N, False, gws.FMT_FP8_E4M3, bt=6.0, seed_id=5, rows_sel=rows_sel, mode=mode)


def test_config5_input_gradient_8192x5632x2048_a_row_in_every_tile():
    # dX = dY * W^T: the [K x N] weight of config 5 read as [N' x K'] = [2048 x 5632], 88 K-steps, one round of 256 tiles
    M, K, N = 8192, 5632, 2048
    dy = (synth.make_activation(51, M, K).float() * 1e-2).to(torch.bfloat16).to(DEV)
    w = synth.make_tensor(52, N, K, bt=6.0, with_grad=False)["w"].to(DEV)
    dx = torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)
    gws.gws_gemm_bf16(dy, w, dx, w_is_nk=True)
    torch.cuda.synchronize()
    rows_sel = tile_rows(M, np.random.default_rng(51))
    check_y(synth.bits(dx), synth.bits(dy), synth.bits(w), True, rows_sel)


def test_linear_mode_errors():
    x = synth.make_activation(4, 200, 96).to(DEV)
    t = synth.make_tensor(4, 96, 160, with_grad=False)
    w, bt = t["w"].to(DEV), t["bt"].to(DEV)
    y = torch.zeros(200, 160, dtype=torch.bfloat16, device=DEV)
    full = gws.TensorDesc(rows=96, cols=160, seed=1, w=w, bt=bt, w_hat=torch.zeros_like(w), scale=torch.zeros(3, 5, device=DEV))
    bare = gws.TensorDesc(rows=96, cols=160, seed=1, w=w, bt=bt)
    with pytest.raises(gws.GwsError) as e:
        gws.gws_linear_fwd_mode(x, full, y, gws.FMT_FP8_E4M3, 0, 1)                         # a retired mode value
    assert e.value.status == 4
    with pytest.raises(gws.GwsError) as e:
        gws.gws_linear_fwd_mode(x, bare, y, gws.FMT_FP8_E4M3, 0, gws.LINEAR_TWO_KERNELS)    # nowhere to put w_hat
    assert e.value.status == 1
    with pytest.raises(gws.GwsError) as e:
        gws.gws_linear_fwd_mode(x, full, y, gws.FMT_FP8_E4M3, 0, 9)
    assert e.value.status == 4
    torch.cuda.synchronize()
    assert (synth.bits(y) == 0).all()                                                        # nothing was launched


def test_large_tile_gemm_random_shapes_and_strides():
    # whole 256 x 256 tiles, few of them (the kernel that splits K), at seeded random shapes: odd and even numbers of
    # K-steps (1 .. 11), padded leading dimensions, both weight layouts; every element against the fp64 GEMM
    rng = np.random.default_rng(2505)
    for case in range(10):
        M, N = 256 * int(rng.integers(1, 4)), 256 * int(rng.integers(1, 4))
        K = 64 * int(rng.integers(1, 12))
        w_is_nk = bool(case & 1)
        padx, padw, pady = (8 * int(rng.integers(0, 3)) for _ in range(3))
        x_full = synth.make_activation(400 + case, M, K + padx).to(DEV)
        wr, wc = (N, K) if w_is_nk else (K, N)
        w_full = synth.make_tensor(400 + case, wr, wc + padw, with_grad=False)["w"].to(DEV)
        y_full = torch.zeros(M, N + pady, dtype=torch.bfloat16, device=DEV)
        x, w, y = x_full[:, :K], w_full[:, :wc], y_full[:, :N]
        gws.gws_gemm_bf16(x, w, y, w_is_nk=w_is_nk)
        torch.cuda.synchronize()
        xb = np.ascontiguousarray(synth.bits(x_full)[:, :K])
        wb = np.ascontiguousarray(synth.bits(w_full)[:, :wc])
        check_y(np.ascontiguousarray(synth.bits(y_full)[:, :N]), xb, wb, w_is_nk)
        assert (synth.bits(y_full)[:, N:] == 0).all(), (case, "padding of Y written")


@pytest.mark.parametrize("w_is_nk", [False, True])
def test_large_tile_gemm_every_number_of_k_steps(w_is_nk):
    # two whole 256 x 256 tiles, 1 .. 14 K-steps of 64: fewer units of K than wavefronts that split it, and several each;
    # every element against fp64 (the large tile's own loop: test_whole_large_tiles_at_every_number_of_k_steps)
    M, N = 256, 512
    for nk in range(1, 15):
        K = 64 * nk
        x = synth.make_activation(700 + nk, M, K).to(DEV)
        wr, wc = (N, K) if w_is_nk else (K, N)
        w = synth.make_tensor(700 + nk, wr, wc, with_grad=False)["w"].to(DEV)
        y = torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)
        gws.gws_gemm_bf16(x, w, y, w_is_nk=w_is_nk)
        torch.cuda.synchronize()
        check_y(synth.bits(y), synth.bits(x), synth.bits(w), w_is_nk)


def run_next_case(M, K, N, w_is_nk, next_rows, next_cols, fmt, idx, step=3, next_pad=0, rows_sel=None, rides=0):
    """gws_gemm_bf16_sample_next: Y against the fp64 GEMM, the forward pass of the next weight, which rides or does not,
    against the oracle."""
    x = synth.make_activation(500 + idx, M, K).to(DEV)
    wr, wc = (N, K) if w_is_nk else (K, N)
    w = synth.make_tensor(500 + idx, wr, wc, with_grad=False)["w"].to(DEV)
    y = torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)
    t = synth.make_tensor(600 + idx, next_rows, next_cols, ld=next_cols + next_pad, with_grad=False)
    nw, nbt = t["w"].to(DEV), t["bt"].to(DEV)
    n_hat = nw.clone()                                     # padding columns must keep these bytes
    nbr, nbc = synth.n_blocks(next_rows, next_cols)
    n_scale = torch.full((nbr, nbc), float("nan"), device=DEV)
    seed = oracle.derive_seed(7, idx)
    nxt = gws.TensorDesc(rows=next_rows, cols=next_cols, ld=next_cols + next_pad, seed=seed, w=nw, w_hat=n_hat, bt=nbt, scale=n_scale)
    assert gws.gws_ride_plan(M, K, N, [nxt], w_is_nk) == rides
    gws.gws_gemm_bf16_sample_next(x, w, y, nxt, fmt, step, w_is_nk=w_is_nk)
    torch.cuda.synchronize()
    check_y(synth.bits(y), synth.bits(x), synth.bits(w), w_is_nk, rows_sel)
    ref_q, ref_s = oracle.sample_fwd(synth.bits(t["w"]), t["bt"].numpy(), fmt, seed, step, cols=next_cols)
    assert (synth.bits(n_hat) == ref_q).all(), ("w_hat of the next weight", idx)
    assert (n_scale.cpu().numpy().view(np.uint32) == ref_s.view(np.uint32)).all(), ("scale of the next weight", idx)
    return y


@pytest.mark.parametrize("fmt", [gws.FMT_BF16, gws.FMT_FP8_E4M3, gws.FMT_FP6_E3M2])
def test_gemm_with_the_next_weight_sampled_alongside(fmt):
    rows_sel = np.array([0, 255, 256, 1279])
    for w_is_nk in (False, True):                                            # 65 tiles: the sampling rides in the same launch
        run_next_case(1280, 64, 3328, w_is_nk, 128, 320, fmt, 8, rows_sel=rows_sel, rides=1)                # next weight of whole 32 x 64 tiles
        run_next_case(1280, 64, 3328, w_is_nk, 256, 1024, fmt, 9, next_pad=8, rows_sel=rows_sel, rides=1)   # of whole 32 x 256 tiles, padded
    run_next_case(768, 192, 1280, False, 128, 320, fmt, 0)                   # a GEMM that splits K: separate launch
    run_next_case(512, 128, 512, True, 256, 1024, fmt, 1, next_pad=8)
    run_next_case(768, 192, 1280, False, 96, 300, fmt, 2, next_pad=4)        # ragged next weight: separate launch
    run_next_case(200, 96, 160, False, 128, 320, fmt, 3)                     # GEMM not on the large tile: separate launch
    run_next_case(256, 64, 256, False, 4096, 4096, fmt, 4)                   # sampling far longer than the GEMM: separate launch


def test_gemm_next_without_idle_compute_units_and_without_next():
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert cus % 16 == 0
    M, N = 256 * 16, 256 * (cus // 16)                                       # exactly one tile per compute unit
    y = run_next_case(M, 64, N, False, 128, 320, gws.FMT_FP8_E4M3, 5, rows_sel=np.array([0, 255, 256, M - 1]))
    # next = None is the plain GEMM
    x = synth.make_activation(505, M, 64).to(DEV)
    w = synth.make_tensor(505, 64, N, with_grad=False)["w"].to(DEV)
    y2 = torch.zeros_like(y)
    gws.gws_gemm_bf16_sample_next(x, w, y2, None, gws.FMT_FP8_E4M3, 0)
    torch.cuda.synchronize()
    assert (synth.bits(y2) == synth.bits(y)).all()


def test_config5_gemm_with_the_next_weight_sampled_alongside():
    rows_sel = tile_rows(8192, np.random.default_rng(6))
    run_next_case(8192, 2048, 5632, False, 2048, 8192, gws.FMT_FP8_E4M3, 6, rows_sel=rows_sel)   # too much to ride: two launches
    run_next_case(8192, 2048, 5632, False, 2048, 5632, gws.FMT_FP8_E4M3, 6, rows_sel=rows_sel, rides=1)   # as long as the last round of tiles
    run_next_case(8192, 2048, 5632, False, 2048, 2048, gws.FMT_FP8_E4M3, 7, rows_sel=rows_sel, rides=1)   # rides beside the last round of tiles


def run_next_list(M, K, N, next_shapes, fmt, idx, step=5, rows_sel=None, w_is_nk=False, rides=0):
    """gws_gemm_bf16_sample_next_n: Y against the fp64 GEMM, every listed weight, of which the first `rides` ride, against the
    oracle's forward pass."""
    x = synth.make_activation(700 + idx, M, K).to(DEV)
    wr, wc = (N, K) if w_is_nk else (K, N)
    w = synth.make_tensor(700 + idx, wr, wc, with_grad=False)["w"].to(DEV)
    y = torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)
    descs, host = [], []
    for k, (r, c) in enumerate(next_shapes):
        ld = (c + 7) // 8 * 8
        t = synth.make_tensor(720 + 10 * idx + k, r, c, ld=ld, with_grad=False)
        nw = t["w"].to(DEV)
        nbr, nbc = synth.n_blocks(r, c)
        descs.append(gws.TensorDesc(rows=r, cols=c, ld=ld, seed=oracle.derive_seed(9, 10 * idx + k), w=nw, w_hat=nw.clone(),
                                    bt=t["bt"].to(DEV), scale=torch.full((nbr, nbc), float("nan"), device=DEV)))
        host.append(t)
    assert gws.gws_ride_plan(M, K, N, descs, w_is_nk) == rides
    gws.gws_gemm_bf16_sample_next_n(x, w, y, descs, fmt, step, w_is_nk=w_is_nk)
    torch.cuda.synchronize()
    check_y(synth.bits(y), synth.bits(x), synth.bits(w), w_is_nk, rows_sel)
    for d, t in zip(descs, host):
        ref_q, ref_s = oracle.sample_fwd(synth.bits(t["w"]), t["bt"].numpy(), fmt, d.seed, step, cols=d.cols)
        assert (synth.bits(d.w_hat) == ref_q).all(), ("w_hat", idx, d.rows, d.cols)
        assert (d.scale.cpu().numpy().view(np.uint32) == ref_s.view(np.uint32)).all(), ("scale", idx, d.rows, d.cols)


@pytest.mark.parametrize("fmt", [gws.FMT_BF16, gws.FMT_FP8_E4M3, gws.FMT_FP6_E3M2])
def test_gemm_with_several_next_weights_sampled_alongside(fmt):
    rows_sel = np.array([0, 255, 256, 2559])
    for w_is_nk in (False, True):
        for lst, rides in [([(128, 512), (64, 256), (96, 768)], 3),                  # all three ride (whole 32 x 256 tiles)
                           ([(128, 512), (96, 300)], 1),                             # the ragged one: separate launch
                           ([(32, 256)] * 5 + [(64, 512)], 4),                       # more than ride at once: the rest after the GEMM
                           ([(96, 320), (128, 512)], 1),                             # first not of whole 32 x 256 tiles: rides alone
                           ([(256, 512), (0, 256), (64, 256)], 1)]:                  # an empty weight in the list
            run_next_list(2560, 64, 4864, lst, fmt, 8, rows_sel=rows_sel, w_is_nk=w_is_nk, rides=rides)
        run_next_list(1280, 64, 3328, [(128, 512), (64, 256), (96, 768)], fmt, 9, rows_sel=rows_sel[:3], w_is_nk=w_is_nk, rides=3)   # under a product of the middle tile
    run_next_list(768, 192, 1280, [(128, 512), (64, 256), (96, 768)], fmt, 0)            # a GEMM that splits K: all separate
    run_next_list(200, 96, 160, [(128, 512), (64, 256)], fmt, 4)                         # of no whole tiles: all separate
    run_next_list(256, 64, 256, [(2048, 2048), (1024, 1024)], fmt, 6)                    # too much to ride beside one short tile


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("fmt", [gws.FMT_BF16, gws.FMT_FP8_E4M3, gws.FMT_FP6_E3M2])
def test_forced_riding_gives_the_same_bytes_for_both_riding_loops(fmt, w_is_nk):
    # include/gws_bench.h, gws_gemm_bf16_ride_probe: riders alone (no GEMM) and beside a GEMM, both riding loops
    step = 8
    t = synth.make_tensor(790, 512, 1280, with_grad=False)
    seed = oracle.derive_seed(3, 790)
    ref_q, ref_s = oracle.sample_fwd(synth.bits(t["w"]), t["bt"].numpy(), fmt, seed, step)
    nw, nbt = t["w"].to(DEV), t["bt"].to(DEV)
    x = synth.make_activation(791, 512, 128).to(DEV)
    w = synth.make_tensor(791, *((768, 128) if w_is_nk else (128, 768)), with_grad=False)["w"].to(DEV)
    for rider in (0, 1):
        for with_gemm in (False, True):
            for extra in (1, 7, 64):
                d = gws.TensorDesc(rows=512, cols=1280, seed=seed, w=nw, w_hat=torch.zeros_like(nw), bt=nbt,
                                   scale=torch.zeros(16, 40, device=DEV))
                y = torch.zeros(512, 768, dtype=torch.bfloat16, device=DEV)
                if with_gemm:
                    gws.gws_gemm_bf16_ride_probe(x, w, y, d, fmt, step, extra, rider, w_is_nk=w_is_nk)
                else:
                    gws.gws_gemm_bf16_ride_probe(None, None, None, d, fmt, step, extra, rider)
                torch.cuda.synchronize()
                assert (synth.bits(d.w_hat) == ref_q).all(), (rider, with_gemm, extra)
                assert (d.scale.cpu().numpy().view(np.uint32) == ref_s.view(np.uint32)).all()
                if with_gemm:
                    check_y(synth.bits(y), synth.bits(x), synth.bits(w), w_is_nk)


# Few rows of X or few tiles: the kernel whose wavefronts split K.  Every tile it has (16 x 16 and 16 x 32 up to 16 rows,
# 32 x 32, 32 x 64, 64 x 64, 128 x 64), one row and one column tile more or less than whole, K of whole and half units of 64, fewer
# units than wavefronts and several per wavefront, padded X and Y; plain and sampled form bit for bit (run_case).
@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("M,K,N", [(1, 64, 32), (16, 96, 64), (17, 128, 96), (4, 1632, 32), (32, 544, 4128), (33, 2080, 1056),
                                   (64, 1024, 2080), (65, 736, 5664), (300, 672, 1056), (511, 1312, 800), (400, 3072, 2048), (500, 3072, 2528)])
def test_gemm_that_splits_k(M, K, N, w_is_nk):
    assert [gws.gws_gemm_form(M, K, N, w_is_nk, k, ldx=K + 8) for k in (0, 1)] == [gws.GEMM_STREAM, gws.GEMM_STREAM_SAMPLE]
    idx = 40 + (M * 7 + K) % 50
    rows_sel = None if M * K * N < 2e7 else np.array(sorted({0, 15 % M, M // 2, M - 1}))
    run_case(M, K, N, w_is_nk, gws.FMT_FP8_E4M3, seed_id=idx, ldx_pad=8, ldy_pad=8, rows_sel=rows_sel, mode=gws.LINEAR_IN_OPERAND)
    run_case(M, K, N, w_is_nk, gws.FMT_FP6_E3M2 if M % 2 else gws.FMT_BF16, seed_id=idx, step=2, rows_sel=rows_sel, mode=gws.LINEAR_IN_OPERAND)
    run_case(M, K, N, w_is_nk, gws.FMT_FP8_E4M3, seed_id=idx, step=4, rows_sel=rows_sel)   # the library's choice between the two forms


# Bands of eight tile rows with one and two more, which are joined to the band before, and with three, which are not: every tile against
# the 64-bit product.
@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("M,K,N,rows", [(257, 96, 768, 9), (290, 128, 448, 10), (321, 96, 672, 11), (513, 192, 256, 17), (576, 96, 416, 18)])
def test_gemm_that_splits_k_of_a_few_tile_rows_over_whole_bands(M, K, N, rows, w_is_nk):
    tile_rows, _, _, parts = gws.gws_gemm_stream_tile(M, K, N, w_is_nk, ldx=K + 8)
    assert -(-M // tile_rows) == rows and parts
    run_case(M, K, N, w_is_nk, gws.FMT_FP8_E4M3, seed_id=63, ldx_pad=8, ldy_pad=8)


# Up to 16 rows the stream kernel keeps eight or sixteen rows and, of [N x K] weights, eight, sixteen or 32 columns of its MFMA tiles: each
# of them, at the edges of the choice (8 and 9 rows, K of 2048, as many eight-column tiles as compute units) and at the smallest.  The
# sampled form, which has one tile for all of these, gives the same bits (run_case).
@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("M,K,N,columns", [(1, 64, 32, 16), (7, 2016, 64, 16), (8, 2048, 2048, 8), (8, 2080, 2080, 16), (9, 2048, 2048, 8), (9, 2016, 96, 16), (16, 2080, 2048, 8),
                                           (16, 2080, 2080, 16), (8, 320, 4128, 32)])
def test_gemm_of_half_an_mfma_tile(M, K, N, columns, w_is_nk):
    assert gws.gws_gemm_stream_tile(M, K, N, w_is_nk, ldx=K + 8)[:2] == (8 if M <= 8 else 16, columns if w_is_nk else 32)
    run_case(M, K, N, w_is_nk, gws.FMT_FP8_E4M3, seed_id=61, ldx_pad=8, ldy_pad=8, mode=gws.LINEAR_IN_OPERAND,
             rows_sel=None if M * K * N < 2e7 else np.array(sorted({0, M // 2, M - 1})))


# Idle compute units fetch the weight into the L2s.  [K x N] (kn workgroups a tile): as many tiles as a quarter and a third of the compute
# units, one tile more than each, and where a round of the XCDs more takes the last of them; [N x K] of 17 to 64 rows (nk): up to half of the
# compute units and one more.  Tiles that do not fill a round, one and two rows of them, half a unit at the end of K, one unit a
# wavefront and many; bit for bit the sampled form's Y, which has no such workgroups (run_case).
@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("M,K,N,kn,nk", [
    (3, 2080, 2048, 3, 0), (16, 1024, 2080, 2, 0), (6, 544, 2560, 2, 0), (6, 544, 2592, 0, 0), (8, 2720, 2720, 0, 0), (4, 608, 4096, 0, 0), (5, 544, 4128, 0, 0),
    (8, 512, 2048, 3, 0), (16, 2048, 512, 3, 0), (24, 1056, 1024, 3, 1), (20, 512, 2048, 3, 1), (64, 1056, 1088, 2, 1), (40, 4096, 256, 3, 1), (20, 544, 3840, 0, 1),
    (20, 544, 4096, 0, 1), (20, 544, 4128, 0, 0)])
def test_gemm_whose_weight_is_fetched_by_idle_compute_units(M, K, N, kn, nk, w_is_nk):
    assert gws.gws_gemm_stream_tile(M, K, N, w_is_nk, ldx=K + 8)[2] == (nk if w_is_nk else kn)
    run_case(M, K, N, w_is_nk, gws.FMT_FP8_E4M3, seed_id=62, ldx_pad=8, ldy_pad=8, mode=gws.LINEAR_IN_OPERAND, rows_sel=np.array(sorted({0, M // 2, M - 1})))


# A large [N x K] weight that the launch before wrote is taken by groups of tiles, kept weights by parts (both in run_case, bit for bit): each
# tile, with and without fetching workgroups, one and four rows of tiles and a last column that is not whole (the query says zeros where
# gws_linear_fwd would sample in the operand load; the two kernels are asked for).
@pytest.mark.parametrize("M,K,N", [(1, 2080, 2048), (16, 1056, 4000), (8, 800, 5280), (33, 2080, 2048), (128, 2080, 2048), (100, 1056, 4000), (203, 2048, 3424)])
def test_gemm_on_a_weight_that_was_just_sampled(M, K, N):
    assert gws.gws_gemm_stream_tile(M, K, N, True, ldx=K + 8)[3] == 1 and gws.gws_gemm_stream_tile(M, K, N, True, ldx=K + 8, sampled=2)[3] == 0
    run_case(M, K, N, True, gws.FMT_FP8_E4M3, seed_id=64, ldx_pad=8, ldy_pad=8, mode=gws.LINEAR_TWO_KERNELS, rows_sel=np.array(sorted({0, M // 2, M - 1})))


def test_riding_under_a_gemm_of_many_k_steps():
    # 182 tiles of 256 x 256: the large tile is the faster one and leaves 74 compute units idle
    assert gws.gws_gemm_form(6656, 1024, 1792) == gws.GEMM_LARGE
    run_next_list(6656, 1024, 1792, [(128, 512), (64, 256), (96, 768)], gws.FMT_FP8_E4M3, 7, rows_sel=np.array([0, 255, 256, 6655]), rides=3)
    # 272 tiles of 256 x 256, 368 of 256 x 192: the narrow tile is the faster one by more than a launch, and nothing rides
    assert gws.gws_gemm_form(4096, 1024, 4352) == gws.GEMM_NARROW
    run_next_list(4096, 1024, 4352, [(128, 512), (64, 256)], gws.FMT_FP8_E4M3, 7, rows_sel=np.array([0, 255, 256, 4095]))


# The middle tile (128 x 128 and 128 x 96 columns) and the large tile with edges: one row and 32 columns more or less than whole tiles, K of
# whole and half steps of 64 (the half step at every place in the rings of loads), padded X and Y; the sampling kernel's Y
# is the same bits.
@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("M,K,N,cols", [(1537, 96, 1696, 96), (1920, 160, 1760, 128), (1600, 256, 2080, 128), (2049, 288, 1312, 96), (2000, 1504, 2016, 128),
                                        (3969, 96, 800, 128), (3969, 320, 928, 128), (3841, 288, 1824, 128)])
def test_middle_tile_gemm(M, K, N, cols, w_is_nk):
    assert gws.gws_gemm_tile(M, K, N, w_is_nk, ldx=K + 8) == (128, cols)
    assert [gws.gws_gemm_form(M, K, N, w_is_nk, k, ldx=K + 8) for k in (0, 1)] == [gws.GEMM_MIDDLE, gws.GEMM_ROWS_SAMPLE]
    run_case(M, K, N, w_is_nk, gws.FMT_FP8_E4M3, seed_id=91, ldx_pad=8, ldy_pad=8, rows_sel=np.array([0, 127, 128, M // 2, M - 1]),
             mode=gws.LINEAR_IN_OPERAND)


# Middle tiles of 128 x 96 (taken here: they and those of 128 x 128 are one round, and theirs is the shorter K-step): a last column
# tile of one wavefront's part, of two thirds of it and whole, a last row tile of 1 row to 128, 1 to 9 K-steps (four stages) whole
# and half; against fp32 on the GPU and bit for bit the sampling kernel's Y, which walks K from end to end as well.
@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("M,N", [(1024, 2304), (1025, 2272), (897, 2336), (1000, 2336)])
def test_middle_tile_of_96_columns_at_every_number_of_k_steps(M, N, w_is_nk):
    for K in [64 * i + 32 * h for i in range(1, 10) for h in (0, 1)]:
        assert gws.gws_gemm_form(M, K, N, w_is_nk) == gws.GEMM_MIDDLE and gws.gws_gemm_tile(M, K, N, w_is_nk) == (128, 96)
        gen = torch.Generator(device=DEV).manual_seed(K)
        x = torch.randn(M, K, generator=gen, device=DEV).to(torch.bfloat16)
        w = (torch.randn(*((N, K) if w_is_nk else (K, N)), generator=gen, device=DEV) * 0.02).to(torch.bfloat16)
        y = torch.zeros(M + 1, N + 8, dtype=torch.bfloat16, device=DEV)
        gws.gws_gemm_bf16(x, w, y[:M, :N], w_is_nk=w_is_nk)
        kn = (w.t().contiguous() if w_is_nk else w).float()
        ref, mag = x.float() @ kn, x.float().abs() @ kn.abs()
        # one rounding to BF16 and two fp32 sums of K terms in different orders
        assert bool(((y[:M, :N].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2 * K * 2.0 ** -24 * mag).all()), K
        assert bool((y[:, N:] == 0).all()) and bool((y[M] == 0).all())
    run_case(M, 352, N, w_is_nk, gws.FMT_FP8_E4M3, seed_id=93, ldx_pad=8, ldy_pad=8, rows_sel=np.array([0, 127, 128, M - 1]), mode=gws.LINEAR_IN_OPERAND)


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("M,K,N", [(8191, 96, 1824), (8193, 512, 1760)] + [(7937, 1024 + 32 * i, 1568) for i in range(1, 13, 2)])
def test_large_tile_gemm_with_edges(M, K, N, w_is_nk):
    assert [gws.gws_gemm_form(M, K, N, w_is_nk, k, ldx=K + 8) for k in (0, 1)] == [gws.GEMM_LARGE_EDGE, gws.GEMM_ROWS_SAMPLE]
    run_case(M, K, N, w_is_nk, gws.FMT_FP8_E4M3, seed_id=92, ldx_pad=8, ldy_pad=8, rows_sel=np.array([0, 255, 256, M // 2, M - 2, M - 1]),
             mode=gws.LINEAR_IN_OPERAND)


@pytest.mark.parametrize("w_is_nk", [False, True])
def test_whole_large_tiles_at_every_number_of_k_steps(w_is_nk):
    # 256 tiles of 256 x 256, 1 to 14 K-steps (the rings' common period is six): against fp32 on the GPU
    for steps in range(1, 15):
        K = 64 * steps
        assert gws.gws_gemm_form(8192, K, 2048, w_is_nk) == gws.GEMM_LARGE
        gen = torch.Generator(device=DEV).manual_seed(steps)
        x = torch.randn(8192, K, generator=gen, device=DEV).to(torch.bfloat16)
        w = (torch.randn(*((2048, K) if w_is_nk else (K, 2048)), generator=gen, device=DEV) * 0.02).to(torch.bfloat16)
        y = torch.zeros(8192, 2048, dtype=torch.bfloat16, device=DEV)
        gws.gws_gemm_bf16(x, w, y, w_is_nk=w_is_nk)
        kn = (w.t().contiguous() if w_is_nk else w).float()
        ref, mag = x.float() @ kn, x.float().abs() @ kn.abs()
        assert bool(((y.float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2 * K * 2.0 ** -24 * mag).all()), steps


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("M,N", [(8192, 2560), (8000, 2336), (4100, 4096)])
def test_narrow_large_tiles_at_every_number_of_k_steps(M, N, w_is_nk):
    # sizes whose 256 x 192 tiles fill the rounds better; whole and ragged edges, K of whole and half steps of 64
    for K in [64 * i + 32 * (i % 2 if i > 1 else 0) for i in range(4, 17)]:
        assert gws.gws_gemm_form(M, K, N, w_is_nk) == gws.GEMM_NARROW
        gen = torch.Generator(device=DEV).manual_seed(K)
        x = torch.randn(M, K, generator=gen, device=DEV).to(torch.bfloat16)
        w = (torch.randn(*((N, K) if w_is_nk else (K, N)), generator=gen, device=DEV) * 0.02).to(torch.bfloat16)
        y = torch.zeros(M, N + 8, dtype=torch.bfloat16, device=DEV)
        gws.gws_gemm_bf16(x, w, y[:, :N], w_is_nk=w_is_nk)
        kn = (w.t().contiguous() if w_is_nk else w).float()
        ref, mag = x.float() @ kn, x.float().abs() @ kn.abs()
        assert bool(((y[:, :N].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2 * K * 2.0 ** -24 * mag).all()), K
        assert bool((y[:, N:] == 0).all())


# Tiles of 256 x 256: a last row tile of 1 and 255 rows, a last column tile of one wavefront, six and eight, 2 to 10 units whole and
# half, the [N x K] weights that K brings here; Y and w_hat bit for bit.  Tiles of 128 x 128 (one workgroup a compute unit and two):
# last row tiles of one wavefront's half and one row, a last column tile of one wavefront, 1 to 11 units whole and half.
@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("tile,M,K,N", [(128, 2240, 96, 1056), (128, 2241, 672, 1120), (128, 3969, 64, 1952), (128, 7937, 160, 416), (256, 4097, 96, 3616),
                                         (256, 7935, 128, 1984), (256, 7937, 160, 2016), (256, 8192, 416, 2048), (256, 4097, 576, 2144), (256, 4001, 608, 2208)])
def test_sampling_in_the_operand_load_of_256_rows_and_by_pairs(tile, M, K, N, w_is_nk):
    assert gws.gws_gemm_tile(M, K, N, w_is_nk, sampled=1, ldx=K + 8) == (tile, tile)
    assert gws.gws_gemm_form(M, K, N, w_is_nk, sampled=1, ldx=K + 8) == gws.GEMM_ROWS_SAMPLE
    for fmt in (gws.FMT_BF16, gws.FMT_FP8_E4M3, gws.FMT_FP6_E3M2):
        run_case(M, K, N, w_is_nk, fmt, seed_id=95, ldx_pad=8, ldy_pad=8, rows_sel=np.array([0, 127, 128, 255, 256, M // 2, M - 1]), mode=gws.LINEAR_IN_OPERAND)


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("M,K,N", [(1500, 160, 1760), (2049, 288, 1312), (1537, 96, 4128), (4160, 64, 544)])
def test_sampling_in_the_operand_load_of_many_rows(M, K, N, w_is_nk):
    assert gws.gws_gemm_form(M, K, N, w_is_nk, sampled=1, ldx=K + 8) == gws.GEMM_ROWS_SAMPLE
    assert gws.gws_gemm_tile(M, K, N, w_is_nk, sampled=1, ldx=K + 8) == (128, 128)
    # a last row tile of 1 to 128 rows, a last column tile of one wavefront, K of whole and half units; Y and w_hat bit for bit
    for fmt in (gws.FMT_BF16, gws.FMT_FP8_E4M3, gws.FMT_FP6_E3M2):
        run_case(M, K, N, w_is_nk, fmt, seed_id=93, ldx_pad=8, ldy_pad=8, rows_sel=np.array([0, 63, 64, M // 2, M - 1]), mode=gws.LINEAR_IN_OPERAND)


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("M", [1, 16, 64])
def test_y_on_top_of_the_weight(M, w_is_nk):
    # a caller with room for w_hat (its own, a workspace, the library's buffer) may be done with w: the weight is then
    # sampled by a kernel of its own, at row counts that otherwise sample in the operand load
    K, N, fmt, step = 1024, 3072, gws.FMT_FP8_E4M3, 6
    assert gws.gws_gemm_form(M, K, N, w_is_nk, sampled=2) == gws.GEMM_STREAM_SAMPLE
    t = synth.make_tensor(95, *((N, K) if w_is_nk else (K, N)), with_grad=False)
    rows, cols = t["w"].shape
    x, bt = synth.make_activation(96, M, K).to(DEV), t["bt"].to(DEV)

    def run(form, on_weight):
        w = t["w"].to(DEV)
        y = w.view(-1)[:M * N].view(M, N) if on_weight else torch.zeros(M, N, dtype=torch.bfloat16, device=DEV)
        d = gws.TensorDesc(rows=rows, cols=cols, seed=4, w=w, bt=bt)
        if form == "hat":
            d.w_hat, d.scale = torch.zeros_like(w), torch.zeros_like(bt)
            gws.gws_linear_fwd(x, d, y, fmt, step, w_is_nk=w_is_nk)
        elif form == "ws":
            ws = torch.zeros(gws.gws_linear_fwd_workspace_bytes(d), dtype=torch.uint8, device=DEV)
            gws.gws_linear_fwd_ws(x, d, y, fmt, step, ws, w_is_nk=w_is_nk)
        else:
            gws.gws_linear_fwd_static(x, d, y, fmt, step, w_is_nk=w_is_nk)
        torch.cuda.synchronize()
        return synth.bits(y)

    ref = run("hat", False)
    for form in ("hat", "ws", "static"):
        assert (run(form, False) == ref).all(), form
        assert (run(form, True) == ref).all(), form


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("M,K,N", [(1, 64, 32), (128, 128, 128), (37, 96, 96), (100, 1024, 128), (256, 256, 256)])
def test_a_product_of_one_tile_in_place(M, K, N, w_is_nk):
    # Y on top of X or of the weight where one workgroup computes all of it: plain, with the weight sampled on its way in,
    # and (up to 128 rows and columns) with it sampled in the operand load
    fmt, step = gws.FMT_FP6_E3M2, 2
    t = synth.make_tensor(97, *((N, K) if w_is_nk else (K, N)), with_grad=False)
    rows, cols = t["w"].shape
    bt, seed = t["bt"].to(DEV), oracle.derive_seed(1, 97)
    xb = synth.make_activation(98, M, K)
    q, _ = oracle.sample_fwd(synth.bits(t["w"]), t["bt"].numpy(), fmt, seed, step)

    def run(on, sampled):
        x, w = xb.to(DEV), t["w"].to(DEV)
        y = (x.view(-1)[:M * N] if on == "x" else w.view(-1)[:M * N]).view(M, N)
        if sampled:
            gws.gws_linear_fwd(x, gws.TensorDesc(rows=rows, cols=cols, seed=seed, w=w, bt=bt), y, fmt, step, w_is_nk=w_is_nk)
        else:
            gws.gws_gemm_bf16(x, w, y, w_is_nk=w_is_nk)
        torch.cuda.synchronize()
        return synth.bits(y)

    for on in ("x", "w"):
        if M * N > (M * K if on == "x" else K * N):
            continue
        check_y(run(on, False), synth.bits(xb), synth.bits(t["w"]), w_is_nk)
        if M <= 128:
            check_y(run(on, True), synth.bits(xb), q, w_is_nk)


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("form,cols,M,K,N", [
    (gws.GEMM_STREAM, 64, 300, 672, 1056), (gws.GEMM_MIDDLE, 96, 1537, 96, 1696), (gws.GEMM_MIDDLE, 96, 1280, 320, 3328),
    (gws.GEMM_MIDDLE, 128, 3969, 96, 800), (gws.GEMM_MIDDLE, 128, 3969, 320, 1824), (gws.GEMM_MIDDLE, 128, 1920, 256, 1792),
    (gws.GEMM_LARGE, 256, 8192, 320, 2048), (gws.GEMM_LARGE, 256, 6656, 832, 1792), (gws.GEMM_LARGE_EDGE, 256, 8191, 96, 1824),
    (gws.GEMM_LARGE_EDGE, 256, 7937, 1056, 1568), (gws.GEMM_NARROW, 192, 8192, 448, 2560), (gws.GEMM_NARROW, 192, 8000, 352, 2336),
    (gws.GEMM_ANY_SHAPE, 128, 300, 32, 416)])
def test_every_gemm_with_padded_operands(form, cols, M, K, N, w_is_nk):
    # X, the weight and Y all in wider buffers, NaN in what the product must not read; against fp32 on the GPU
    padx, padw, pady = 24, 40, 8
    gen = torch.Generator(device=DEV).manual_seed(M + K)
    wr, wc = (N, K) if w_is_nk else (K, N)
    x = torch.full((M, K + padx), float("nan"), dtype=torch.bfloat16, device=DEV)
    w = torch.full((wr, wc + padw), float("nan"), dtype=torch.bfloat16, device=DEV)
    y = torch.zeros(M, N + pady, dtype=torch.bfloat16, device=DEV)
    x[:, :K] = torch.randn(M, K, generator=gen, device=DEV)
    w[:, :wc] = torch.randn(wr, wc, generator=gen, device=DEV) * 0.02
    assert gws.gws_gemm_form(M, K, N, w_is_nk, ldx=K + padx, ldw=wc + padw) == form
    assert gws.gws_gemm_tile(M, K, N, w_is_nk, ldx=K + padx, ldw=wc + padw)[1] == cols
    gws.gws_gemm_bf16(x[:, :K], w[:, :wc], y[:, :N], w_is_nk=w_is_nk)
    kn = (w[:, :wc].t().contiguous() if w_is_nk else w[:, :wc]).float()
    xf = x[:, :K].float()
    ref, mag = xf @ kn, xf.abs() @ kn.abs()
    # one rounding to BF16 and two fp32 sums of K terms in different orders
    assert bool(((y[:, :N].float() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2 * K * 2.0 ** -24 * mag).all())
    assert bool((y[:, N:] == 0).all())


@pytest.mark.parametrize("M,K,N", [(4224, 96, 2048), (4096, 160, 2176), (4001, 544, 2144)])
def test_sampling_in_the_operand_load_on_the_tiles_of_any_shape(M, K, N):
    # the [N x K] weights of 513 to 768 tiles of 128 x 128, which keep the kernel of the 32x32x16 MFMA and K-steps of 32:
    # Y bit for bit that of the GEMM behind the sampling kernel, which takes another (16x16x32, steps of 64)
    assert [gws.gws_gemm_form(M, K, N, True, k, ldx=K + 8) for k in (0, 1)] == [gws.GEMM_NARROW, gws.GEMM_ANY_SHAPE_SAMPLE]
    for fmt in (gws.FMT_BF16, gws.FMT_FP8_E4M3, gws.FMT_FP6_E3M2):
        run_case(M, K, N, True, fmt, seed_id=94, ldx_pad=8, ldy_pad=8, rows_sel=np.array([0, 127, 128, M // 2, M - 1]), mode=gws.LINEAR_IN_OPERAND)


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("M,K,N,ldx,plain", [(130, 96, 160, 1 << 23, gws.GEMM_MIDDLE), (100, 160, 96, 1 << 24, gws.GEMM_ANY_SHAPE), (256, 320, 256, 1 << 24, gws.GEMM_LARGE)])
def test_rows_of_x_far_apart(M, K, N, ldx, plain, w_is_nk):
    # leading dimensions beyond the 32-bit lane offsets of some kernels: the others take over, and the two forms of the
    # sampled linear still give the same bits
    assert [gws.gws_gemm_form(M, K, N, w_is_nk, k, ldx=ldx) for k in (0, 1)] == [plain, gws.GEMM_ANY_SHAPE_SAMPLE]
    fmt, step, seed = gws.FMT_FP8_E4M3, 3, oracle.derive_seed(0, 99)
    t = synth.make_tensor(99, *((N, K) if w_is_nk else (K, N)), with_grad=False)
    rows, cols = t["w"].shape
    xs = synth.make_activation(99, M, K)
    x = torch.empty(M, ldx, dtype=torch.bfloat16, device=DEV)[:, :K]
    x.copy_(xs)
    w, bt = t["w"].to(DEV), t["bt"].to(DEV)
    d = gws.TensorDesc(rows=rows, cols=cols, seed=seed, w=w, bt=bt, w_hat=torch.zeros_like(w), scale=torch.zeros_like(bt))
    y = [torch.zeros(M, N, dtype=torch.bfloat16, device=DEV) for _ in range(2)]
    gws.gws_linear_fwd_mode(x, d, y[0], fmt, step, gws.LINEAR_TWO_KERNELS, w_is_nk=w_is_nk)
    gws.gws_linear_fwd_mode(x, d, y[1], fmt, step, gws.LINEAR_IN_OPERAND, w_is_nk=w_is_nk)
    torch.cuda.synchronize()
    q, _ = oracle.sample_fwd(synth.bits(t["w"]), t["bt"].numpy(), fmt, seed, step)
    check_y(synth.bits(y[0]), synth.bits(xs), q, w_is_nk)
    assert (synth.bits(y[0]) == synth.bits(y[1])).all()


@pytest.mark.parametrize("w_is_nk", [False, True])
@pytest.mark.parametrize("fmt", [gws.FMT_BF16, gws.FMT_FP8_E4M3, gws.FMT_FP6_E3M2])
@pytest.mark.parametrize("tile,M,K,N", [(16, 1, 64, 32), (16, 5, 96, 64), (16, 16, 992, 160), (32, 17, 96, 32), (64, 40, 544, 96), (64, 200, 96, 96), (64, 3000, 96, 160),
                                        (128, 3000, 160, 2208), (128, 2900, 352, 992), (64, 5, 96, 8288), (64, 16, 64, 8224), (64, 40, 544, 8224),
                                        (64, 755, 96, 2592), (128, 1700, 64, 3104), (16, 5, 1696, 16416), (16, 16, 1664, 16416), (64, 218, 8576, 2336)])
def test_blocks_sampled_by_one_and_by_pairs(tile, M, K, N, fmt, w_is_nk):
    assert gws.gws_gemm_tile(M, K, N, w_is_nk, sampled=1)[0] == tile
    # up to 16 rows two blocks a step, with more than one workgroup a compute unit one, more rows one, many two again: one, two,
    # three blocks of K and odd numbers of them (half a step at the end), wavefronts without any, a shard; w_hat, scale and Y to the bits of the sampling kernel and the
    # plain product
    r, c = (N, K) if w_is_nk else (K, N)
    t = synth.make_tensor(60 + M % 7, r, c, device=DEV, bt=3.0 if M == 40 else None)     # b_t = 3: blocks beyond the hardware cast
    x = synth.make_activation(61 + M % 5, M, K, device=DEV)
    nb = synth.n_blocks(r, c)
    shard = dict(rows=r, cols=c, seed=9, row0=64, col0=96)
    one, two = (gws.TensorDesc(**shard, w=t["w"], bt=t["bt"], w_hat=torch.zeros_like(t["w"]), scale=torch.zeros(*nb, device=DEV)) for _ in range(2))
    y, ref = (torch.zeros(M, N, dtype=torch.bfloat16, device=DEV) for _ in range(2))
    gws.gws_linear_fwd_mode(x, one, y, fmt, 4, gws.LINEAR_IN_OPERAND, w_is_nk=w_is_nk)
    gws.gws_sample_fwd([two], fmt, 4)
    gws.gws_gemm_bf16(x, two.w_hat, ref, w_is_nk=w_is_nk)
    torch.cuda.synchronize()
    assert torch.equal(one.w_hat.view(torch.int16), two.w_hat.view(torch.int16)) and torch.equal(one.scale, two.scale)
    assert torch.equal(y.view(torch.int16), ref.view(torch.int16))
