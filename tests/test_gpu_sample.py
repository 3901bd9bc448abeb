"""GPU parity of gws_sample_fwd / gws_sample_bwd / gws_noise_packed against the CPU
oracle, through the C ABI.  Bit-exact for noise codes, sampled weights, scales and dW;
1e-5 relative (+ cancellation floor) for dL/db_t."""
import numpy as np
import pytest
import torch

import oracle
import paper_2505_11170_amd as gws
from paper_2505_11170_amd import synth
from gpu_util import CANCELLATION_SHARE, DEV, assert_dbt_close, ensure_built, gpu_backward, gpu_forward

pytestmark = pytest.mark.gpu

FMTS = [gws.FMT_BF16, gws.FMT_FP8_E4M3, gws.FMT_FP6_E3M2]


@pytest.fixture(scope="module", autouse=True)
def _lib():
    ensure_built()


def check_forward(items, fmt, step):
    outs, _ = gpu_forward(items, fmt, step)
    for it, (w_hat, scale) in zip(items, outs):
        if it["rows"] == 0 or it["cols"] == 0:
            continue
        wb = synth.bits(it["w"])
        ref_w, ref_s = oracle.sample_fwd(wb, it["bt"].cpu().numpy(), fmt, it["seed"], step, cols=it["cols"],
                                         row0=it.get("row0", 0), col0=it.get("col0", 0))
        assert (scale.view(np.uint32) == ref_s.view(np.uint32)).all(), ("scale", it["rows"], it["cols"])
        bad = np.argwhere(w_hat != ref_w)
        assert len(bad) == 0, ("w_hat", it["rows"], it["cols"], fmt, bad[:5])
    return outs


def check_backward(items, step, dw_mode="copy"):
    outs, keep = gpu_backward(items, step, dw_mode)
    needed = 0
    for it, (dw, dbt) in zip(items, outs):
        if it["rows"] == 0 or it["cols"] == 0:
            continue
        gb = synth.bits(it["g"])
        ref_dw, ref_dbt, asum = oracle.sample_bwd(gb, np.asarray(it["scale"]), it["seed"], step, cols=it["cols"],
                                                  row0=it.get("row0", 0), col0=it.get("col0", 0))
        if dw_mode == "copy":
            assert (dw == ref_dw).all()
        needed += assert_dbt_close(dbt, ref_dbt, asum, (it["rows"], it["cols"]))
    return needed


def make_items(shapes, bt=None, base=0, user_seed=0, ld_pad=0):
    items = []
    for i, (r, c) in enumerate(shapes):
        ld = ((c + 7) // 8) * 8 + ld_pad
        t = synth.make_tensor(base + i, r, c, bt=bt, ld=ld)
        items.append(dict(w=t["w"], bt=t["bt"], g=t["g"], rows=r, cols=c, seed=oracle.derive_seed(user_seed, base + i)))
    return items


def test_noise_codes_bit_exact():
    for (rows, cols, row0, col0, seed, step) in [(64, 64, 0, 0, 1, 0), (37, 45, 0, 0, 2 ** 63 + 5, 2 ** 40 + 3),
                                                 (768, 768, 0, 0, oracle.derive_seed(0, 0), 0),
                                                 (40, 72, 96, 64, 77, 9)]:
        out = torch.zeros(rows, (cols + 7) // 8, dtype=torch.int32, device=DEV)
        gws.gws_noise_packed(out, rows, cols, seed, step, row0=row0, col0=col0)
        torch.cuda.synchronize()
        _, ref = oracle.noise(rows, cols, seed, step, row0=row0, col0=col0)
        assert (out.cpu().numpy().view(np.uint32) == ref).all()


def test_config1_single_768x768_e4m3_forward():
    t = synth.make_tensor(0, 768, 768, bt=6.0, with_grad=False)
    item = dict(w=t["w"], bt=t["bt"], rows=768, cols=768, seed=oracle.derive_seed(0, 0))
    outs = check_forward([item], gws.FMT_FP8_E4M3, 0)
    assert np.isfinite(outs[0][1]).all()


@pytest.mark.parametrize("fmt", FMTS)
def test_forward_ragged_shapes_all_formats(fmt):
    shapes = [(96, 160), (70, 45), (33, 257), (32, 32), (1, 1), (31, 7), (257, 600), (64, 512), (40, 264)]
    check_forward(make_items(shapes), fmt, 3)


def test_forward_row_padding_is_never_written():
    items = make_items([(45, 70), (64, 100)], ld_pad=16)
    outs, keep = gpu_forward(items, gws.FMT_FP8_E4M3, 1)
    for it, (w_hat, _) in zip(items, outs):
        wb = synth.bits(it["w"])
        assert (w_hat[:, it["cols"]:] == wb[:, it["cols"]:]).all()
    check_forward(items, gws.FMT_FP8_E4M3, 1)


def test_many_tensors_span_several_launches_and_skip_empty_ones():
    shapes = [(32 * (1 + i % 5), 32 * (1 + (3 * i) % 7)) for i in range(95)]
    shapes[7] = (0, 64)
    shapes[50] = (64, 0)
    items = make_items(shapes, base=100)
    for it in items:
        if it["rows"] == 0 or it["cols"] == 0:
            it["w"] = torch.zeros(1, 8, dtype=torch.bfloat16)
            it["g"] = torch.zeros(1, 8, dtype=torch.bfloat16)
            it["bt"] = torch.zeros(1, 1)
    outs = check_forward(items, gws.FMT_FP6_E3M2, 2)
    for it, (_, s) in zip(items, outs):
        it["scale"] = s if it["rows"] and it["cols"] else np.zeros((1, 1), np.float32)
    check_backward(items, 2)


@pytest.mark.parametrize("dw_mode", ["copy", "none", "alias"])
def test_backward_ragged_shapes(dw_mode):
    shapes = [(96, 160), (70, 45), (33, 257), (32, 32), (1, 1), (257, 600)]
    items = make_items(shapes, base=20)
    outs, _ = gpu_forward(items, gws.FMT_BF16, 11)
    for it, (_, s) in zip(items, outs):
        it["scale"] = s
    check_backward(items, 11, dw_mode)


def test_backward_uses_the_forward_noise():
    # g = w_hat - w (BF16 target, b_t = 4): then sum(g .* R) = s * sum(R^2) up to rounding,
    # which only holds if backward regenerates exactly the forward R.
    rows = cols = 128
    t = synth.make_tensor(30, rows, cols, bt=4.0)
    seed = oracle.derive_seed(3, 30)
    item = dict(w=t["w"], bt=t["bt"], rows=rows, cols=cols, seed=seed)
    (w_hat, scale), = gpu_forward([item], gws.FMT_BF16, 5)[0]
    r, _ = oracle.noise(rows, cols, seed, 5)
    g = synth.from_bits(oracle.bf16_add_n(w_hat.ravel(), (synth.bits(t["w"]).ravel() ^ 0x8000)).reshape(rows, cols))
    item_b = dict(g=g, scale=scale, rows=rows, cols=cols, seed=seed)
    (dw, dbt), = gpu_backward([item_b], 5)[0]
    r2 = (r.astype(np.float64) ** 2).reshape(4, 32, 4, 32).sum(axis=(1, 3))
    approx = -np.log(2.0) * scale.astype(np.float64) ** 2 * r2
    assert np.allclose(dbt, approx, rtol=0.05)
    # and with the wrong step the correlation is gone
    (_, dbt_wrong), = gpu_backward([item_b], 6)[0]
    assert np.abs(dbt_wrong).mean() < 0.3 * np.abs(dbt).mean()


def test_shard_origin_reproduces_full_tensor_noise():
    rows, cols = 128, 256
    t = synth.make_tensor(40, rows, cols)
    seed = 4242
    full = dict(w=t["w"], bt=t["bt"], rows=rows, cols=cols, seed=seed)
    (w_full, s_full), = gpu_forward([full], gws.FMT_FP8_E4M3, 7)[0]
    r0, c0 = 64, 96
    sub = dict(w=t["w"][r0:, c0:c0 + 128].contiguous(), bt=t["bt"][r0 // 32:, c0 // 32:c0 // 32 + 4].contiguous(),
               rows=rows - r0, cols=128, seed=seed, row0=r0, col0=c0)
    (w_sub, s_sub), = check_forward([sub], gws.FMT_FP8_E4M3, 7)
    assert (w_sub == w_full[r0:, c0:c0 + 128]).all()
    assert (s_sub == s_full[r0 // 32:, c0 // 32:c0 // 32 + 4]).all()


def test_large_extents_and_origins():
    # long thin tensors (2^20 rows or columns) and shard origins near the 32-bit limits of the
    # noise counter: row index and column-group index wrap the same way on both sides
    for rows, cols in ((32, 1 << 20), (1 << 20, 32)):
        t = synth.make_tensor(70, rows, cols, with_grad=True)
        item = dict(w=t["w"], bt=t["bt"], g=t["g"], rows=rows, cols=cols, seed=oracle.derive_seed(5, 70))
        outs = check_forward([item], gws.FMT_FP8_E4M3, 2 ** 40 + 7)
        item["scale"] = outs[0][1]
        check_backward([item], 2 ** 40 + 7)
    t = synth.make_tensor(71, 64, 128, with_grad=False)
    for row0, col0 in ((2 ** 32 - 64 - 32, 0), (0, 8 * (2 ** 32 - 1) - 128 - 8 * 3), (2 ** 31, 2 ** 33)):
        col0 -= col0 % 32
        item = dict(w=t["w"], bt=t["bt"], rows=64, cols=128, seed=99, row0=row0, col0=col0)
        check_forward([item], gws.FMT_BF16, 1)


def test_determinism_and_step_dependence():
    items = make_items([(256, 512)], base=50)
    a = gpu_forward(items, gws.FMT_FP8_E4M3, 4)[0][0][0]
    _ = gpu_forward(items, gws.FMT_FP8_E4M3, 5)[0][0][0]
    b = gpu_forward(items, gws.FMT_FP8_E4M3, 4)[0][0][0]
    assert (a == b).all() and (a != _).mean() > 0.05


def test_edge_values_zero_blocks_negative_zero_tiny_and_extreme_bt():
    rows, cols = 64, 128
    t = synth.make_tensor(60, rows, cols)
    w = t["w"].clone()
    w[:32, :32] = 0.0                         # all-zero block
    w[0, 0] = -0.0
    w[:32, 32:64] *= 2.0 ** -60               # tiny but inside the supported domain
    w[40, 70] = -0.0
    wb = synth.bits(w).copy()
    wb[33, 1] = 0x0001                        # BF16 subnormal elements inside a normal block
    wb[34, 2] = 0x8040
    w = synth.from_bits(wb)
    bt = t["bt"].clone()
    bt[0, 2] = 60.0                           # noise far below an ulp
    bt[0, 3] = 1.0                            # huge noise: exercises saturation of the cast
    bt[1, 0] = 0.0
    bt[1, 1] = 2.5
    bt[1, 2] = 12.75
    for fmt in FMTS:
        check_forward([dict(w=w, bt=bt, rows=rows, cols=cols, seed=9)], fmt, 0)


def test_config2_gpt2_124m_all_linears_fwd_bwd_3_steps():
    shapes = [(s.rows, s.cols) for s in synth.gpt2_124m_shapes()]
    assert len(shapes) == 48 and sum(r * c for r, c in shapes) == 84_934_656
    items = make_items(shapes)
    needed = 0
    for step in range(3):
        outs = check_forward(items, gws.FMT_FP8_E4M3, step)
        for it, (_, s) in zip(items, outs):
            it["scale"] = s
        needed += check_backward(items, step)
    print(f"config 2: blocks needing the cancellation term of the db_t tolerance: {needed} of {3 * 82944}")
    assert needed <= CANCELLATION_SHARE * 3 * 82944


def test_copy_tiles_moves_exactly_the_tensor():
    # the measurement aid shares the forward pass's launch shape: every element copied once, padding untouched
    shapes = [(768, 768), (40, 50), (33, 257), (0, 64), (96, 320)]
    descs, keep = [], []
    for i, (r, c) in enumerate(shapes):
        ld = (c + 7) // 8 * 8 + 8
        t = synth.make_tensor(900 + i, r, c, ld=ld, with_grad=False)
        w = t["w"].to(DEV)
        out = torch.full_like(w, 7.0)
        descs.append(gws.TensorDesc(rows=r, cols=c, seed=0, w=w, w_hat=out, ld=ld))
        keep.append((w, out, c))
    gws.gws_copy_tiles(descs)
    torch.cuda.synchronize()
    for w, out, c in keep:
        assert torch.equal(out[:, :c].view(torch.int16), w[:, :c].view(torch.int16))
        assert (out[:, c:] == 7.0).all()


def test_block_absmax_is_exact():
    shapes = [(768, 768), (40, 50), (33, 257), (0, 64), (96, 320), (1, 1)]
    descs, keep = [], []
    for i, (r, c) in enumerate(shapes):
        ld = (c + 7) // 8 * 8 + 8
        t = synth.make_tensor(920 + i, r, c, ld=ld, with_grad=False)
        w = t["w"].clone()
        w[:, c:] = 1.0e30                                   # padding must not enter the maximum
        if r >= 33 and c >= 40:
            w[32, 39] = -3.0                                # a negative maximum, in an edge position of its block
        nbr, nbc = synth.n_blocks(r, c)
        out = torch.full((nbr, nbc), float("nan"), device=DEV)
        descs.append(gws.TensorDesc(rows=r, cols=c, seed=0, w=w.to(DEV), scale=out, ld=ld))
        keep.append((w, out, r, c))
    gws.gws_block_absmax(descs)
    torch.cuda.synchronize()
    for w, out, r, c in keep:
        if r == 0 or c == 0:
            continue
        wv = w[:, :c].float().abs().numpy()
        nbr, nbc = synth.n_blocks(r, c)
        ref = np.array([[wv[bi * 32:bi * 32 + 32, bj * 32:bj * 32 + 32].max() for bj in range(nbc)] for bi in range(nbr)],
                       dtype=np.float32)
        assert np.array_equal(out.cpu().numpy(), ref), (r, c)


@pytest.mark.parametrize("seed", [1, 2, 3])
def test_random_mixes_of_many_small_and_ragged_tensors(seed):
    # more tensors than one launch holds, shapes from one element to several workgroup tiles wide:
    # exercises the workgroup -> tensor lookup, the grouping of column tiles and every edge case of the tile code
    rng = np.random.default_rng(seed)
    n = 70
    shapes = [(int(rng.integers(1, 200)), int(rng.integers(1, 1400))) for _ in range(n)]
    shapes[5] = (0, 40)
    shapes[17] = (64, 0)
    shapes[23] = (32, 256)
    shapes[40] = (33, 1025)
    items = make_items(shapes, 1000 + 100 * seed, user_seed=seed)
    fmt = FMTS[seed % 3]
    outs = check_forward(items, fmt, step=seed)
    for it, (_, scale) in zip(items, outs):
        it["scale"] = scale
    check_backward(items, step=seed, dw_mode="copy" if seed % 2 else "alias")


def test_launch_shape_choices_give_the_same_bytes():
    # include/gws_bench.h: the kernel variant (any-shape kernel with four and eight wavefronts a SIMD, whole-tile
    # kernel) and the column tiles a workgroup walks are launch-shape choices; forward and backward results may
    # not depend on them.  Whole-tile tensors (the whole-tile kernels run, forward at one column tile a workgroup:
    # the any-shape kernel at more), a ragged one mixed in (the launch falls back to the
    # any-shape kernel), a shard origin, and the bitwidth left per block.
    shapes = [(64, 512), (96, 1280), (32, 256), (128, 768)]
    for mix in (shapes, shapes + [(40, 300)]):
        descs = []
        for i, (r, c) in enumerate(mix):
            t = synth.make_tensor(1500 + i, r, c, ld=(c + 7) // 8 * 8, device=DEV)
            nbr, nbc = synth.n_blocks(r, c)
            descs.append(gws.TensorDesc(rows=r, cols=c, ld=t["w"].stride(0), seed=oracle.derive_seed(6, i), row0=32 * i, col0=64 * i,
                                        w=t["w"], w_hat=torch.zeros_like(t["w"]), bt=t["bt"], scale=torch.zeros(nbr, nbc, device=DEV),
                                        g=t["g"], dw=t["g"], dbt=torch.zeros(nbr, nbc, device=DEV)))
        outs = lambda: [x.clone() for d in descs for x in (d.w_hat, d.scale, d.dbt)]
        gws.gws_sample_fwd(descs, gws.FMT_FP8_E4M3, 4)
        gws.gws_sample_bwd(descs, 4)
        torch.cuda.synchronize()
        ref = outs()
        for variant in (0, 1, 2):
            for per_x in (1, 2, 3, 5):
                for d in descs:
                    d.w_hat.zero_(), d.scale.zero_(), d.dbt.zero_()
                gws.gws_sample_fwd_tuned(descs, gws.FMT_FP8_E4M3, 4, variant, per_x)
                gws.gws_sample_bwd_tuned(descs, 4, variant, per_x)
                torch.cuda.synchronize()
                for k, (a, b) in enumerate(zip(outs(), ref)):
                    # forward outputs bit for bit; dL/db_t too: both kernels add in the same order
                    assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), (len(mix), variant, per_x, k)
    # and the reference itself is the oracle's
    d = descs[1]
    ref_q, ref_s = oracle.sample_fwd(synth.bits(d.w), d.bt.cpu().numpy(), oracle.FMT_FP8_E4M3, d.seed, 4, cols=d.cols, row0=d.row0, col0=d.col0)
    assert (synth.bits(d.w_hat) == ref_q).all()


@pytest.mark.parametrize("shape", [(768, 768), (32, 256), (96, 300), (1000, 1000), (1, 8)])
def test_one_weight_alone(shape):
    # a small call of one tensor has kernels of its own (descriptor in the kernel's arguments); whole tiles and ragged
    items = make_items([shape], base=880)
    (_, items[0]["scale"]), = check_forward(items, gws.FMT_FP8_E4M3, 6)
    check_backward(items, 6, dw_mode="alias")
    check_backward(items, 6)


@pytest.mark.parametrize("rows", [1, 7, 8, 9, 16, 17, 24, 25, 31, 40, 49, 88])
def test_every_number_of_rows_of_a_last_block(rows):
    # at an edge the noise is drawn for as many groups of eight rows as exist, two together or one alone; the columns whole
    # tiles, a part of one and of a group
    for fmt in FMTS:
        items = make_items([(rows, 256), (rows, 300), (rows, 5)], base=1800 + rows)
        for it, (_, scale) in zip(items, check_forward(items, fmt, 6)):
            it["scale"] = scale
    check_backward(items, 6, dw_mode="alias")
    check_backward(items, 6)


def test_large_calls_give_the_bytes_of_small_ones():
    # 7 x 33.6 MB in rows of 8200 bytes (not whole cache lines: ordinary stores, streaming loads) and in rows of 8320
    # (whole lines, streaming both ways) against the same weights one at a time (ordinary accesses)
    for ld in (4104, 4160):
        gen = torch.Generator(device=DEV).manual_seed(ld)
        w = [(torch.randn(4100, ld, generator=gen, device=DEV) * 0.02).to(torch.bfloat16) for _ in range(7)]
        bt = 4 + 5 * torch.rand(129, 129, generator=gen, device=DEV)

        def descs():
            return [gws.TensorDesc(rows=4100, cols=4100, ld=ld, seed=30 + i, w=w[i], bt=bt, w_hat=torch.zeros_like(w[i]), scale=torch.zeros_like(bt),
                                   g=w[i], dw=torch.zeros_like(w[i]), dbt=torch.zeros_like(bt)) for i in range(7)]
        a, b = descs(), descs()
        gws.gws_sample_fwd(a, gws.FMT_FP6_E3M2, 3)
        gws.gws_sample_bwd(a, 3)
        for d in b:
            gws.gws_sample_fwd([d], gws.FMT_FP6_E3M2, 3)
            gws.gws_sample_bwd([d], 3)
        torch.cuda.synchronize()
        for x, y in zip(a, b):
            assert torch.equal(x.w_hat.view(torch.int16), y.w_hat.view(torch.int16)) and torch.equal(x.scale, y.scale)
            assert torch.equal(x.dw[:, :4100].view(torch.int16), x.g[:, :4100].view(torch.int16)) and torch.equal(x.dbt, y.dbt)


@pytest.mark.parametrize("ld,rows", [((1 << 27) - 8, 40), (1 << 27, 40), ((1 << 27) - 8, 32), (1 << 27, 32)])
def test_rows_longer_than_the_lane_offsets_reach(ld, rows):
    """Full tiles are addressed by 32-bit lane offsets where ld < 2^27; longer rows go the way of the edges, same bits: the longest row
    of the first way and the shortest of the second, by the kernels for any shape (40 rows) and for whole tiles."""
    cols, step = 512, 5
    t = synth.make_tensor(1700, rows, cols, device=DEV)
    far = {k: torch.empty(rows * ld, dtype=torch.bfloat16, device=DEV).view(rows, ld) for k in ("w", "w_hat")}
    far["w"][:, :cols] = t["w"]
    nb = synth.n_blocks(rows, cols)
    out = []
    for w, w_hat, g in ((t["w"], torch.zeros_like(t["w"]), t["g"]), (far["w"], far["w_hat"], None)):
        d = gws.TensorDesc(rows=rows, cols=cols, ld=w.stride(0), seed=3, w=w, w_hat=w_hat, bt=t["bt"], scale=torch.zeros(*nb, device=DEV))
        gws.gws_sample_fwd([d], gws.FMT_FP8_E4M3, step)
        if g is None:
            far["w"][:, :cols] = t["g"]
            g = far["w"]
        d.g, d.dw, d.dbt = g, g, torch.zeros(*nb, device=DEV)
        gws.gws_sample_bwd([d], step)
        torch.cuda.synchronize()
        out.append([w_hat[:, :cols].contiguous().view(torch.int16), d.scale.view(torch.int32), d.dbt.view(torch.int32)])
    for a, b in zip(*out):
        assert torch.equal(a, b)


# One weight alone in a call has an argument block of its own, and above 2048 workgroup tiles of 32 x 256 its tiles are dealt out: at that line
# and over it, whole tiles and ragged ones, rounds of 128 workgroups with and without a rest, every kind of pass; the same bits as
# beside a second weight.
@pytest.mark.parametrize("rows,cols", [(4096, 4096), (4128, 4096), (4100, 4090), (32 * 2049, 256), (65600, 40), (70, 262200)])
def test_one_large_weight_alone_and_beside_another(rows, cols):
    nbr, nbc = synth.n_blocks(rows, cols)
    ld = (cols + 7) // 8 * 8
    gen = torch.Generator(device=DEV).manual_seed(rows)
    w = (torch.randn(rows, ld, device=DEV, generator=gen) * 0.02).to(torch.bfloat16)
    g = (torch.randn(rows, ld, device=DEV, generator=gen) * 1e-3).to(torch.bfloat16)
    bt = 4 + 5 * torch.rand(nbr, nbc, device=DEV, generator=gen)
    small = dict(w=w[:32, :32].contiguous(), bt=bt[:1, :1].contiguous())
    small_out = lambda: dict(w_hat=torch.zeros_like(small["w"]), scale=torch.ones_like(small["bt"]), g=small["w"], dw=torch.zeros_like(small["w"]), dbt=torch.zeros_like(small["bt"]))
    ldc = [(cols * 6 + 7) // 8 + 1 & ~1, ld]

    def run(beside):
        outs = []

        def descs(**out):
            outs.extend(out.values())
            return [gws.TensorDesc(rows=rows, cols=cols, ld=ld, seed=5, w=w, bt=bt, g=g, **out)] + \
                   ([gws.TensorDesc(rows=32, cols=32, ld=32, seed=6, **small, **small_out())] if beside else [])
        scale = lambda: torch.ones_like(bt)
        gws.gws_sample_fwd(descs(w_hat=torch.zeros_like(w), scale=scale()), gws.FMT_FP8_E4M3, 3)
        gws.gws_sample_fwd_basis(descs(w_hat=torch.zeros_like(w), scale=scale()), gws.BASIS_UNIFORM_BF16, gws.FMT_BF16, 3)
        for fmt, l in ((gws.FMT_FP6_E3M2, ldc[0]), (gws.FMT_FP8_E4M3, ldc[1])):
            codes, xs = torch.zeros(rows * l, dtype=torch.uint8, device=DEV), torch.zeros(nbr * nbc, dtype=torch.uint8, device=DEV)
            outs.extend((codes, xs))
            other = [gws.MxOut(torch.zeros(32 * 32, dtype=torch.uint8, device=DEV), torch.zeros(1, dtype=torch.uint8, device=DEV), 24 if fmt == gws.FMT_FP6_E3M2 else 32)]
            gws.gws_sample_fwd_mx(descs(scale=scale()), [gws.MxOut(codes, xs, l)] + (other if beside else []), fmt, 3)
        gws.gws_sample_bwd(descs(scale=scale(), dw=torch.zeros_like(g), dbt=torch.zeros_like(bt)), 3)
        gws.gws_sample_bwd_basis(descs(scale=scale(), dw=torch.zeros_like(g), dbt=torch.zeros_like(bt)), gws.BASIS_BOX_MULLER, 3)
        torch.cuda.synchronize()
        return outs
    for i, (a, b) in enumerate(zip(run(False), run(True))):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), i
