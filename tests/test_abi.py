"""Host-side checks of the C ABI: the library loads, exports every symbol that
include/gws.h declares, validates arguments before any launch, and derives seeds
like the oracle.  No GPU work is issued here."""
import ctypes
import os
import re

import pytest

import oracle
from paper_2505_11170_amd import binding
from paper_2505_11170_amd.binding import _CBitwidth, _CMxOut, _CTensor

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(binding.library_path()):
        from paper_2505_11170_amd.build import build_library
        build_library()
    return binding.load_library()


def declared_symbols(header="gws.h"):
    text = open(os.path.join(ROOT, "include", header)).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(gws_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = declared_symbols()
    assert {"gws_sample_fwd", "gws_sample_bwd", "gws_linear_fwd"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n
    assert set(names) == set(binding.EXPORTS)
    assert lib.gws_version() >= 1
    # the method's header lists no measurement aid; those live in their own header
    bench = declared_symbols("gws_bench.h")
    assert set(bench) == set(binding.BENCH_EXPORTS) and not set(bench) & set(names)
    for n in bench:
        assert hasattr(lib, n), n


def test_derive_seed_matches_oracle(lib):
    for u, t in [(0, 0), (0, 1), (1, 0), (0xDEADBEEF12345678, 0x1_00000002), (2 ** 64 - 1, 2 ** 64 - 1)]:
        assert binding.gws_derive_seed(u, t) == oracle.derive_seed(u, t)


def _t(**kw):
    c = _CTensor()
    for k, v in kw.items():
        setattr(c, k, v)
    return c


def test_argument_validation_launches_nothing(lib):
    OK, NULL, SHAPE, ALIGN, FORMAT, LAUNCH, ALIAS = range(7)
    fake = 0x10000  # never dereferenced: every case below fails validation first
    base = dict(w=fake, w_hat=fake + 0x100000, bt=fake, scale=fake, g=fake, dw=None, dbt=fake,
                rows=64, cols=64, ld=64, row0=0, col0=0, seed=1)

    def fwd(fmt=1, **over):
        arr = (_CTensor * 1)(_t(**{**base, **over}))
        return lib.gws_sample_fwd(arr, 1, fmt, 0, None)

    def bwd(**over):
        arr = (_CTensor * 1)(_t(**{**base, **over}))
        return lib.gws_sample_bwd(arr, 1, 0, None)

    assert lib.gws_sample_fwd(None, 0, 1, 0, None) == OK          # empty list
    assert lib.gws_sample_fwd(None, 1, 1, 0, None) == NULL
    assert lib.gws_sample_fwd(None, -1, 1, 0, None) == SHAPE
    assert fwd(rows=0) == OK and fwd(cols=0) == OK and bwd(rows=0) == OK   # empty tensors are skipped
    assert fwd(w=None) == NULL and fwd(w_hat=None) == NULL and fwd(bt=None) == NULL and fwd(scale=None) == NULL
    assert fwd(fmt=3) == FORMAT and fwd(fmt=-1) == FORMAT
    assert fwd(ld=60) == SHAPE and fwd(ld=56) == SHAPE and fwd(rows=-1) == SHAPE and fwd(cols=2 ** 31) == SHAPE
    assert fwd(row0=16) == SHAPE and fwd(col0=8) == SHAPE and fwd(row0=-32) == SHAPE
    assert fwd(w=fake + 2) == ALIGN and fwd(w_hat=fake + 0x100008) == ALIGN and fwd(bt=fake + 1) == ALIGN
    assert fwd(w_hat=fake) == ALIAS and fwd(w_hat=fake + 64) == ALIAS
    assert bwd(g=None) == NULL and bwd(dbt=None) == NULL and bwd(scale=None) == NULL
    assert bwd(g=fake + 4) == ALIGN and bwd(dw=fake + 32) == ALIAS
    assert bwd(ld=63) == SHAPE
    assert lib.gws_noise_packed(None, 4, 4, 0, 0, 0, 0, None) == NULL
    assert lib.gws_noise_packed(fake, 4, 4, 0, 4, 0, 0, None) == SHAPE
    assert lib.gws_noise_packed(None, 0, 4, 0, 0, 0, 0, None) == OK
    # linear: shape rules
    wdesc = (_CTensor * 1)(_t(**base))
    assert lib.gws_linear_fwd(fake, 8, 32, 32, wdesc, 0, 1, 0, fake, 64, None) == SHAPE      # K mismatch
    assert lib.gws_linear_fwd(fake, 8, 64, 64, wdesc, 0, 9, 0, fake, 64, None) == FORMAT
    assert lib.gws_linear_fwd_mode(fake, 8, 64, 64, wdesc, 0, 1, 0, fake, 64, 4, None) == FORMAT    # no such mode
    assert lib.gws_linear_fwd_mode(fake, 8, 64, 64, wdesc, 0, 1, 0, fake, 64, -1, None) == FORMAT
    assert lib.gws_linear_fwd_mode(fake, 8, 64, 64, wdesc, 0, 1, 0, fake, 64, 1, None) == FORMAT    # a retired mode value
    assert lib.gws_linear_fwd_mode(fake, 0, 64, 64, wdesc, 0, 1, 0, fake, 64, 3, None) == OK        # empty
    # linear with w_hat staged in a workspace: the workspace is checked like any buffer
    need = lib.gws_linear_fwd_workspace_bytes(wdesc)
    assert need == 64 * 64 * 2 + 4 * 4 and lib.gws_linear_fwd_workspace_bytes(None) == 0
    ws = fake + 0x900000
    lin = (fake + 0x300000, 8, 64, 64, wdesc, 0, 1, 0, fake + 0x500000, 64)
    assert lib.gws_linear_fwd_ws(*lin, None, need, None) == NULL
    assert lib.gws_linear_fwd_ws(*lin, ws + 16, need, None) == ALIGN
    assert lib.gws_linear_fwd_ws(*lin, ws, need - 1, None) == SHAPE
    assert lib.gws_linear_fwd_ws(*lin, fake, need, None) == ALIAS                                  # workspace on w
    assert lib.gws_linear_fwd_ws(*lin, fake + 0x500000, need, None) == ALIAS                       # workspace on y
    assert lib.gws_linear_fwd_ws(fake, 0, 64, 64, wdesc, 0, 1, 0, fake, 64, None, 0, None) == OK   # empty
    # the allocation-free form: same argument rules; a weight beyond the library's staging buffer is refused
    TOO_LARGE = 7
    assert lib.gws_linear_fwd_static(None, 8, 64, 64, wdesc, 0, 1, 0, fake + 0x500000, 64, None) == NULL
    assert lib.gws_linear_fwd_static(fake + 0x300000, 8, 32, 32, wdesc, 0, 1, 0, fake + 0x500000, 64, None) == SHAPE
    assert lib.gws_linear_fwd_static(fake, 0, 64, 64, wdesc, 0, 1, 0, fake, 64, None) == OK        # empty
    big = (_CTensor * 1)(_t(**{**base, "rows": 4096, "cols": 4096 + 32, "ld": 4096 + 32}))         # 33 MiB of w_hat
    assert lib.gws_linear_fwd_workspace_bytes(big) > 32 << 20
    assert lib.gws_linear_fwd_static(fake + 0x300000, 8, 4096, 4096, big, 0, 1, 0, fake + 0x500000, 4128, None) == TOO_LARGE
    assert lib.gws_gemm_bf16(fake, 8, 48, 48, fake, 64, 64, 0, fake, 64, None) == SHAPE      # K % 32
    assert lib.gws_gemm_bf16(None, 8, 64, 64, fake, 64, 64, 0, fake, 64, None) == NULL
    assert lib.gws_gemm_bf16(fake, 0, 64, 64, fake, 64, 64, 0, fake, 64, None) == OK         # empty
    # GEMM with the next weight's sampling: the next weight is checked like gws_sample_fwd's, and may not
    # overlap the GEMM's operands
    nxt = (_CTensor * 1)(_t(**base))
    gemm = (fake, 256, 64, 64, fake + 0x400000, 256, 256, 0, fake + 0x800000, 256)
    assert lib.gws_gemm_bf16_sample_next(*gemm, nxt, 9, 0, None) == FORMAT
    assert lib.gws_gemm_bf16_sample_next(*gemm, (_CTensor * 1)(_t(**{**base, "bt": None})), 1, 0, None) == NULL
    assert lib.gws_gemm_bf16_sample_next(*gemm, (_CTensor * 1)(_t(**{**base, "w_hat": fake + 0x400000})), 1, 0, None) == ALIAS
    assert lib.gws_gemm_bf16_sample_next(*gemm, (_CTensor * 1)(_t(**{**base, "w_hat": fake + 0x800040})), 1, 0, None) == ALIAS
    assert lib.gws_gemm_bf16_sample_next(fake, 256, 48, 48, fake + 0x400000, 256, 256, 0, fake + 0x800000, 256, nxt, 1, 0, None) == SHAPE
    assert lib.gws_gemm_bf16_sample_next(None, 256, 64, 64, fake + 0x400000, 256, 256, 0, fake + 0x800000, 256, nxt, 1, 0, None) == NULL
    for s in range(8):
        assert lib.gws_status_string(s)


def test_descriptor_fields_that_are_no_64_bit_whole_numbers():
    # as ctypes treats its fields: too large wraps (and the library refuses what comes out), no whole number is a TypeError
    d = binding.TensorDesc(rows=2 ** 63 + 64, cols=64, ld=64, seed=-1)
    c = binding._marshal([d, binding.TensorDesc(rows=32, cols=64, ld=64, seed=2 ** 64 + 5)])
    assert (c[0].rows, c[0].cols, c[0].seed) == (64 - 2 ** 63, 64, 2 ** 64 - 1) and (c[1].rows, c[1].seed, c[1].w) == (32, 5, None)
    with pytest.raises(binding.GwsError) as e:
        binding._check(binding.load_library().gws_sample_fwd(binding._marshal([d]), 1, 1, 0, None), "gws_sample_fwd")
    assert e.value.status == 2
    for bad in (1.5, None, "64"):
        with pytest.raises(TypeError):
            binding._marshal([binding.TensorDesc(rows=bad, cols=64, ld=64, seed=1)])


def test_queries_of_the_chosen_kernel(lib):
    # host functions: what rides and which kernel a call takes, by layout; without a device for 256 compute units
    nxt = [binding.TensorDesc(rows=512, cols=512, ld=512, seed=1)]
    assert [binding.gws_ride_plan(1536, 320, 4096, nxt, w_is_nk=nk) for nk in (False, True)] == [1, 0]
    assert lib.gws_ride_plan(1536, 320, 4096, binding._marshal(nxt), 1) == 1           # the [K x N] weight's
    assert binding.gws_gemm_form(1024, 48, 64) == 0 and binding.gws_gemm_form(0, 64, 64) == 0   # what the GEMM refuses, and an empty one
    assert binding.gws_gemm_form(4, 5632, 2048, w_is_nk=True) == binding.GEMM_STREAM
    assert binding.gws_gemm_form(8192, 2048, 5632) == binding.GEMM_LARGE
    assert [binding.gws_gemm_form(m, 2048, 5632, sampled=2) for m in (16, 8192)] == [binding.GEMM_STREAM_SAMPLE, binding.GEMM_LARGE]
    assert binding.gws_gemm_form(2**30, 64, 2**30) == 0 or binding.gws_gemm_tile(2**30, 64, 2**30)[0] > 0   # more tiles than a grid has
    tile = binding.gws_gemm_tile                                                      # and the part of Y that a workgroup makes
    assert tile(1024, 48, 64) == (0, 0) and tile(1024, 32, 64) == (128, 128)
    assert [tile(4, 5632, 2048, nk) for nk in (True, False)] == [(16, 16), (16, 32)] and tile(4, 5632, 2048, sampled=1) == (16, 32)
    assert [tile(8192, 2048, n) for n in (5632, 2560)] == [(256, 256), (256, 192)]
    assert [tile(2048, 2048, 2048), tile(1024, 768, 2304)] == [(128, 128), (128, 96)]
    assert [tile(m, 2048, 2048, sampled=1) for m in (2048, 8192)] == [(128, 128), (256, 256)]
    launch = binding.gws_gemm_stream_tile                                             # rows, columns, workgroups that fetch, parts
    assert [launch(m, 2048, 2048, True)[:2] for m in (8, 9, 17)] == [(8, 8), (16, 8), (32, 32)] and launch(8192, 2048, 5632) == (0, 0, 0, 0)
    assert [launch(8, 2048, n)[2] for n in (2048, 2560, 2592)] == [3, 2, 0] and [launch(20, 544, n, True)[2] for n in (4096, 4128)] == [1, 0]
    # [K x N], two tile rows and more: parts, unless the columns are a multiple of 512 beyond 2048 and the tiles one round of the compute units
    assert [launch(100, 2048, n)[3] for n in (2048, 2304, 2336, 2560, 2592, 3072, 5600)] == [1, 1, 1, 0, 1, 0, 1] and launch(132, 4096, 5632)[3] == 1
    assert [launch(16, 2048, n)[3] for n in (2304, 2336)] == [0, 0] and [launch(100, 2048, n, True)[3] for n in (96, 2560)] == [0, 1]
    # the launch before writes the weight: [N x K] of 8 MB and more, up to four tile rows, by groups
    after = lambda m, k, n, nk=True: (launch(m, k, n, nk)[3], launch(m, k, n, nk, sampled=2)[3])
    assert [after(64, 5632, 2048), after(128, 2048, 2048), after(16, 5632, 2048), after(203, 2048, 3424)] == [(1, 0)] * 4
    assert [after(129, 2048, 2048), after(128, 2048, 2016), after(261, 2336, 5952), after(64, 5632, 2048, False)] == [(1, 1)] * 4
    assert launch(64, 5632, 2048, True)[:3] == launch(64, 5632, 2048, True, sampled=2)[:3] and launch(16, 768, 768, True, sampled=2) == (0, 0, 0, 0)
    wide = binding.TensorDesc(rows=4096, cols=4096, ld=4096, seed=1)
    assert binding.gws_linear_bwd_w_form(wide, 512) == binding.BWD_W_WIDE and binding.gws_linear_bwd_w_form(wide, 63) == 0


# Under products of the middle and the narrow tile, what was faster by more than 8 % (MI355X): the weights riding under the 256-tile, or
# sampled behind the product's own kernel.
@pytest.mark.parametrize("M,K,N,nk,weights,rides", [
    (1280, 1024, 3328, False, [(1024, 1024)], 0), (1280, 768, 3328, False, [(256, 512)], 0), (2048, 1024, 2304, False, [(1024, 512)], 0),
    (2304, 1088, 2304, False, [(768, 2304)], 0), (2304, 704, 2048, False, [(512, 256)], 0), (3840, 512, 1280, True, [(512, 512)], 0),
    (1280, 128, 4864, False, [(256, 256)], 1), (5120, 128, 1536, False, [(256, 512)], 1), (3072, 128, 2048, True, [(256, 256)], 1),
    (1280, 192, 4608, False, [(256, 256), (2304, 256)], 2)])
def test_weights_ride_where_that_measured_faster(lib, M, K, N, nk, weights, rides):
    descs = [binding.TensorDesc(rows=r, cols=c, ld=c, seed=1) for r, c in weights]
    assert binding.gws_gemm_form(M, K, N, nk) in (binding.GEMM_MIDDLE, binding.GEMM_NARROW)
    assert binding.gws_ride_plan(M, K, N, descs, w_is_nk=nk) == rides


# Weight gradient: the form that was fastest by more than 8 % when every one was timed (MI355X, operands in turn from copies beyond the
# L2), rows on cache lines and off; parts that the workspace has room for.
@pytest.mark.parametrize("tokens,rows,cols,parts,on,off", [
    (512, 512, 512, 0, "32", "32"), (4096, 512, 256, 8, "32", None), (4096, 768, 768, 8, "64", None), (2048, 1024, 1024, 4, "64", "64"),
    (4096, 768, 3072, 7, "96", "96"), (4096, 768, 3072, 0, "96", "96"), (2048, 768, 3072, 4, "96", "96"), (8192, 768, 3072, 0, "96", "96"),
    (2048, 2048, 2048, 4, "128x128", "128x128"), (2816, 1280, 2304, 0, "128x128", "128x128"), (1920, 4352, 512, 3, "128x128", "128x128"),
    (8192, 2048, 2048, 0, "128x128", "128x128"), (8192, 2048, 2048, 4, "128x128", None), (4032, 256, 256, 7, "32", "32"),
    (2816, 1280, 2304, 5, "parts", "parts"), (3584, 2048, 2816, 2, "parts", "parts"), (5760, 3072, 2048, 2, "parts", "parts"),
    (8192, 512, 512, 8, None, "parts"), (8128, 1792, 256, 8, None, "parts"), (1024, 2048, 4096, 0, "narrow", "narrow"), (512, 4096, 4096, 0, "wide", "wide")])
def test_the_form_of_a_weight_gradient_is_the_one_that_measured_fastest(lib, tokens, rows, cols, parts, on, off):
    forms = {"32": binding.BWD_W_PIECES_32, "64": binding.BWD_W_PIECES_64, "96": binding.BWD_W_PIECES_96, "128x128": binding.BWD_W_PIECES_128_128,
             "parts": binding.BWD_W_SPLIT + parts, "narrow": binding.BWD_W_NARROW, "wide": binding.BWD_W_WIDE}
    d = binding.TensorDesc(rows=rows, cols=cols, ld=cols, seed=1)
    for on_lines, name in ((True, on), (False, off)):
        if name is not None:
            assert binding.gws_linear_bwd_w_form(d, tokens, parts * rows * cols * 4, on_lines=on_lines) == forms[name]
    # without the flag the query is of an ordinary call: contiguous operands, rows on lines
    assert lib.gws_linear_bwd_w_form(binding._marshal([d]), tokens, parts * rows * cols * 4) == binding.gws_linear_bwd_w_form(d, tokens, parts * rows * cols * 4)


def test_pieces_of_a_weight_gradient_are_not_given_up_for_longer_sums():
    # off the lines, where four or eight sums an element are as fast as three or seven parts
    for tokens, rows, cols, parts in [(1920, 4352, 512, 3), (4032, 256, 256, 7)]:
        assert binding.gws_linear_bwd_w_form(binding.TensorDesc(rows=rows, cols=cols, ld=cols, seed=1), tokens, parts * rows * cols * 4, on_lines=False) < binding.BWD_W_SPLIT


def test_bitwidth_and_mx_entry_points_validate_before_any_launch(lib):
    OK, NULL, SHAPE, ALIGN, FORMAT, LAUNCH, ALIAS = range(7)
    fake = 0x10000  # never dereferenced: every case below fails validation first
    base = dict(w=fake, w_hat=fake + 0x100000, bt=fake, scale=fake, g=fake, dw=None, dbt=fake,
                rows=64, cols=64, ld=64, row0=0, col0=0, seed=1)
    bw = (_CBitwidth * 1)()
    bw[0].b_init, bw[0].b_target, bw[0].lam, bw[0].layer_blocks = 6.0, 4.0, 0.0, 0

    def arr(**over):
        return (_CTensor * 1)(_t(**{**base, **over}))

    assert lib.gws_sample_fwd_bi(arr(), 1, None, 1, 0, None) == NULL           # no bitwidth settings
    assert lib.gws_sample_fwd_bi(None, 0, None, 1, 0, None) == OK              # empty list
    assert lib.gws_sample_fwd_bi(arr(), 1, bw, 7, 0, None) == FORMAT
    assert lib.gws_sample_fwd_bi(arr(bt=None), 1, bw, 1, 0, None) == NULL
    assert lib.gws_sample_bwd_bi(arr(bt=None), 1, bw, 0, None) == NULL         # backward needs b_i here
    assert lib.gws_sample_bwd_bi(arr(bt=fake + 2), 1, bw, 0, None) == ALIGN
    bw[0].layer_blocks = -1
    assert lib.gws_sample_bwd_bi(arr(), 1, bw, 0, None) == SHAPE
    assert lib.gws_sample_bwd_bi(arr(rows=0), 1, bw, 0, None) == SHAPE         # checked for every tensor, empty or not

    def mx(fmt=1, codes=fake + 0x200000, xscale=fake, ldc=64, **over):
        o = (_CMxOut * 1)()
        o[0].codes, o[0].xscale, o[0].ldc = codes, xscale, ldc
        return lib.gws_sample_fwd_mx(arr(**over), o, 1, fmt, 0, None)

    assert mx(fmt=0) == FORMAT and mx(fmt=3) == FORMAT                         # MX exists for FP8 and FP6 only
    assert mx(codes=None) == NULL and mx(xscale=None) == NULL and mx(w=None) == NULL
    assert mx(w_hat=None, rows=0) == OK                                        # w_hat is not used; empty tensors are skipped
    assert mx(ldc=56) == SHAPE and mx(ldc=68) == SHAPE                         # FP8: >= cols, multiple of 8
    assert mx(fmt=2, ldc=46) == SHAPE and mx(fmt=2, ldc=49) == SHAPE           # FP6: >= 48 bytes, even
    assert mx(codes=fake + 0x200004) == ALIGN and mx(fmt=2, ldc=48, codes=fake + 0x200001) == ALIGN
    assert mx(codes=fake + 128) == ALIAS                                       # codes inside w
    assert lib.gws_sample_fwd_mx(arr(), None, 1, 1, 0, None) == NULL


def test_missing_library_fails_loudly(monkeypatch, tmp_path):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_LIB_PATH", str(tmp_path / "libgws.so"))
    with pytest.raises(RuntimeError, match="no CPU or PyTorch fallback"):
        binding.load_library()
