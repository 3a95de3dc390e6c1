"""The row-tile projections (up to 256 rows in one tile, K in steps of 64, loads straight into LDS): edges of
the row blocks, K ranges shorter than the pipeline, uneven K parts, the divided last round, sums that do not
depend on the tile, and which kernel a few rows run on.  Against the fp64 product; one bf16 rounding (2^-8 with
a safety factor) plus the fp32 accumulation error."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _inputs(m, n, k, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    a = torch.empty(m, k, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    w = torch.empty(n, k, dtype=torch.bfloat16, device="cuda").normal_(0.0, k ** -0.5, generator=gen)
    return gen, a, w, a.double() @ w.double().t().contiguous()


def _close(got, ref, extra=0.0):
    got, ref = got.double(), ref
    assert torch.isfinite(got).all()
    bound = 2.0 ** -8 * ref.abs() + 1e-5 * ref.abs().max() + extra
    worst = float(((got - ref).abs() - bound).max())
    assert worst <= 0, worst


ROWS = [1, 8, 9, 16, 17, 31, 32, 33, 56, 64, 65, 96, 97, 128, 129, 160, 192, 193, 224, 255, 256]


@pytest.mark.parametrize("m", ROWS)
def test_rows_times_steps_and_parts(m):
    from paper_2604_14889_amd import binding as M
    # K steps of 64: one, fewer than the LDS stages, more; K parts that do not divide the steps evenly
    for n, k, split in ((128, 64, 1), (256, 128, 1), (384, 192, 3), (128, 256, 2), (256, 320, 5), (640, 448, 2), (256, 1152, 4), (256, 2368, 2)):
        gen, a, w, ref = _inputs(m, n, k, m * 100 + k)
        bias = torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
        need = M.ms_gemm_workspace_bytes(m, n, k, split)
        assert m <= 16 or need == (split * m * n * 4 if split > 1 else 0)
        ws = torch.full((max(need, 16),), 255, dtype=torch.uint8, device="cuda")     # NaN wherever a part is not written
        cut = 128 if n > 128 else n
        outs = [torch.full((m, c), float("nan"), dtype=torch.bfloat16, device="cuda") for c in ((cut, n - cut) if n > cut else (n,))]
        M.ms_gemm_bf16(a, w, bias, outs, split, ws)
        _close(torch.cat(outs, dim=1), ref + bias.double())


@pytest.mark.parametrize("m", [1, 7, 8, 9, 16])
def test_few_rows_with_enough_units_for_the_chip(m):
    """Up to 16 rows run here where the K parts or the columns fill the chip (else on the few-row kernel)."""
    from paper_2604_14889_amd import binding as M
    for n, k, split in ((4608, 3584, 7), (3584, 2304, 8), (37888, 512, 1), (33024, 192, 1)):
        gen, a, w, ref = _inputs(m, n, k, m * 7 + k)
        need = M.ms_gemm_workspace_bytes(m, n, k, split)
        for ws in (torch.full((max(need, 16),), 255, dtype=torch.uint8, device="cuda"), None):
            if ws is None and split > 1:
                continue
            out = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device="cuda")
            M.ms_gemm_bf16(a, w, None, [out], split, ws)
            _close(out, ref)
    tok = torch.full((m,), -1, dtype=torch.int32, device="cuda")
    M.ms_lm_head_argmax_bf16(a, w, tok, torch.empty(M.ms_lm_head_argmax_workspace_bytes(m, n, k), dtype=torch.uint8, device="cuda"))
    top = ref.topk(2, dim=1)
    clear = top.values[:, 0] - top.values[:, 1] > 1e-4 * ref.abs().max()
    assert (tok.long() == top.indices[:, 0])[clear].all() and clear.sum() >= 0.8 * m


@pytest.mark.parametrize("m,n,k", [(64, 66560, 512), (100, 33408, 1024), (200, 33408, 512), (256, 66048, 640), (17, 65664 + 128, 512)])
def test_divided_last_round_and_whole_tiles_without_workspace(m, n, k):
    """More tiles than fit the chip at once: the few left over are divided over K."""
    from paper_2604_14889_amd import binding as M
    gen, a, w, ref = _inputs(m, n, k, m + n)
    need = M.ms_gemm_workspace_bytes(m, n, k, 1)
    assert need > 0
    for ws in (torch.full((need,), 255, dtype=torch.uint8, device="cuda"), None):
        out = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device="cuda")
        M.ms_gemm_bf16(a, w, None, [out], 1, ws)
        _close(out, ref)
    # SwiGLU over the same product: gate and up rows interleaved in blocks of 32 (33408 columns at K up to 1024 are one
    # round of wide tiles with either; K parts of every height with SwiGLU: test_gate_up_takes_wide_tiles_where_they_are_ahead)
    blocks = ref.view(m, n // 64, 2, 32)
    gate, up = blocks[:, :, 0].reshape(m, n // 2), blocks[:, :, 1].reshape(m, n // 2)
    want = gate * torch.sigmoid(gate) * up
    for ws in (torch.full((need,), 255, dtype=torch.uint8, device="cuda"), None):
        act = torch.full((m, n // 2), float("nan"), dtype=torch.bfloat16, device="cuda")
        M.ms_gemm_swiglu_bf16(a, w, act, ws)
        _close(act, want, 2e-5 * (gate.abs() + 1) * (up.abs() + 1))


@pytest.mark.parametrize("m", [17, 56, 96, 128, 192, 224])
def test_greedy_token_and_norm_tail(m):
    from paper_2604_14889_amd import binding as M
    gen, a, w, ref = _inputs(m, 1280, 704, m)
    out = torch.full((m,), -1, dtype=torch.int32, device="cuda")
    M.ms_lm_head_argmax_bf16(a, w, out, torch.empty(M.ms_lm_head_argmax_workspace_bytes(m, 1280, 704), dtype=torch.uint8, device="cuda"))
    top = ref.topk(2, dim=1)
    clear = top.values[:, 0] - top.values[:, 1] > 1e-4 * ref.abs().max()
    assert clear.sum() > 0.8 * m and (out.long() == top.indices[:, 0])[clear].all()
    # the norm behind the product: the same bits as the product, then the norm
    g = torch.empty(1280, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    h = torch.empty(m, 1280, device="cuda").normal_(generator=gen)
    ws = torch.empty(M.ms_gemm_add_rmsnorm_workspace_bytes(m, 1280, 704, 2), dtype=torch.uint8, device="cuda")
    h1, h2 = h.clone(), h.clone()
    o1, o2, d = (torch.empty(m, 1280, dtype=torch.bfloat16, device="cuda") for _ in range(3))
    M.ms_gemm_add_rmsnorm_bf16(a, w, h1, g, 1e-6, o1, 2, ws)
    M.ms_gemm_bf16(a, w, None, [d], 2, ws)
    M.ms_add_rmsnorm(h2, d, g, 1e-6, o2)
    assert torch.equal(h1, h2) and torch.equal(o1.view(torch.int16), o2.view(torch.int16))
    _close(d, ref)


@pytest.mark.parametrize("m", [128, 129, 256])
def test_wide_outputs_that_fill_the_chip_on_either_kernel(m):
    """65664 columns are more than two row-tile units per compute unit: above 128 rows the 256 x 256 tiles take them."""
    from paper_2604_14889_amd import binding as M
    n, k = 65664, 128
    gen, a, w, ref = _inputs(m, n, k, m)
    need = M.ms_gemm_workspace_bytes(m, n, k, 1)
    for ws in (torch.full((max(need, 16),), 255, dtype=torch.uint8, device="cuda"), None):
        out = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device="cuda")
        M.ms_gemm_bf16(a, w, None, [out], 1, ws)
        _close(out, ref)


@pytest.mark.parametrize("m", [1, 7, 8, 9, 16, 17, 64, 128])
def test_equal_weight_rows_give_equal_logits(m):
    """Greedy decoding over logits takes the lowest of equal maxima: copies of a weight row have to give the same
    bits in whatever column tile they are.  Above 16 rows the last, partly filled round of tiles is divided over K
    when there is a workspace for it, so only the full rounds agree there."""
    from paper_2604_14889_amd import binding as M
    tiles = torch.cuda.get_device_properties(0).multi_processor_count
    for n, k in ((128 * (tiles + 40), 1024), (128 * (2 * tiles + 7), 640)):
        gen, a, w, _ = _inputs(m, 128, k, m + k)
        w = w.repeat(n // 128, 1)                            # every column tile holds the same rows
        need = M.ms_gemm_workspace_bytes(m, n, k, 1)
        for ws in (torch.empty(max(need, 16), dtype=torch.uint8, device="cuda"), None):
            out = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device="cuda")
            M.ms_gemm_bf16(a, w, None, [out], 1, ws)
            full = n if m <= 16 or ws is None else n // 128 // tiles * tiles * 128
            same = out.view(torch.int16).view(m, n // 128, 128)[:, :full // 128]
            assert torch.equal(same, same[:, :1].expand_as(same)), (m, n, k)
            if full == n:
                tok = torch.empty(m, dtype=torch.int32, device="cuda")
                M.ms_argmax_rows(out, n, tok)
                assert int(tok.max()) < 128


ROUTES = [
    # M, N, K, split_k: plain products with one launch on the few-row kernel, or on the row tiles where that is ahead
    (1, 3584, 3584, 8, "skinny_mfma_bf16"), (8, 3584, 3584, 8, "skinny_mfma_bf16"), (9, 3584, 3584, 8, "gemm_rows_bf16"),
    (7, 4096, 4096, 8, "skinny_mfma_bf16"), (7, 6144, 4096, 4, "skinny_mfma_bf16"), (8, 4096, 4096, 8, "gemm_rows_bf16"),
    (3, 8192, 8192, 8, "skinny_mfma_bf16"), (4, 8192, 8192, 8, "gemm_rows_bf16"),
    (4, 4608, 3584, 7, "skinny_mfma_bf16"), (5, 4608, 3584, 7, "gemm_rows_bf16"),
    (8, 65536, 1024, 1, "skinny_mfma_bf16"), (9, 65536, 1024, 1, "gemm_rows_bf16"), (8, 65536, 2048, 1, "skinny_mfma_bf16"),
    (1, 65536, 3072, 1, "gemm_rows_bf16"),
]


@pytest.mark.parametrize("m,n,k,split,kernel", ROUTES)
def test_few_rows_run_on_the_kernel_that_is_ahead(m, n, k, split, kernel):
    from paper_2604_14889_amd import binding as M
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the rule was measured on 256 compute units")
    gen, a, w, ref = _inputs(m, n, k, m + n + k)
    ws = torch.full((max(M.ms_gemm_workspace_bytes(m, n, k, split), 16),), 255, dtype=torch.uint8, device="cuda")
    out = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device="cuda")
    M.ms_gemm_bf16(a, w, None, [out], split, ws)
    assert M.ms_gemm_last_kernel() == kernel
    _close(out, ref)


@pytest.mark.parametrize("m", [1, 8, 17, 33, 100, 161, 256, 257, 300])
@pytest.mark.parametrize("shift", [4, 8])
def test_destinations_on_8_byte_boundaries(m, shift):
    """Results leave as 16-byte pieces of whole lines where the destination allows it, as 8-byte ones otherwise;
    the elements around a destination keep their values."""
    from paper_2604_14889_amd import binding as M
    from paper_2604_14889_amd.binding import interleave_gate_up
    n, k = 384, 192
    gen, a, w, ref = _inputs(m, n, k, m + shift)
    bufs = [torch.full((m * c + 16,), 77.0, dtype=torch.bfloat16, device="cuda") for c in (128, 256)]
    outs = [b[shift:shift + m * c].view(m, c) for b, c in zip(bufs, (128, 256))]
    assert outs[0].data_ptr() % 16 == (8 if shift == 4 else 0)
    M.ms_gemm_bf16(a, w, None, outs, 1, torch.empty(max(16, M.ms_gemm_workspace_bytes(m, n, k, 1)), dtype=torch.uint8, device="cuda"))
    _close(torch.cat(outs, dim=1), ref)
    gate, up = ref[:, :192], ref[:, 192:]
    act = torch.full((m * 192 + 16,), 77.0, dtype=torch.bfloat16, device="cuda")
    M.ms_gemm_swiglu_bf16(a, interleave_gate_up(w[:192].contiguous(), w[192:].contiguous()), act[shift:shift + m * 192].view(m, 192))
    _close(act[shift:shift + m * 192].view(m, 192), gate * torch.sigmoid(gate) * up, 1e-5)
    for b, c in ((bufs[0], 128), (bufs[1], 256), (act, 192)):
        assert (b[:shift] == 77).all() and (b[shift + m * c:] == 77).all()


@pytest.mark.parametrize("m", [1, 8, 9, 16, 17, 32, 33, 64, 65, 96, 97, 128, 129, 192, 193, 256])
@pytest.mark.parametrize("inter,k", [(16384 + 64, 64), (18944, 704), (20480, 192), (20480 + 64, 2048), (24576, 640)])
def test_gate_up_in_one_round_of_wide_tiles(m, inter, k):
    """More 128-column tiles than compute units, at most as many of 160 or 192: odd numbers of groups, a last tile
    that is partly past N, K shorter and longer than the pipeline, rows a multiple of 4 KB apart."""
    from paper_2604_14889_amd import binding as M
    gen, a, w, ref = _inputs(m, 2 * inter, k, m + inter + k)
    buf = torch.full((m * inter + 8,), 77.0, dtype=torch.bfloat16, device="cuda")
    out = buf[:m * inter].view(m, inter)
    M.ms_gemm_swiglu_bf16(a, M.interleave_gate_up(w[:inter].contiguous(), w[inter:].contiguous()), out)
    assert M.ms_gemm_last_kernel() == "gemm_rows_bf16"     # the family: which of its kernels, the K parts tell (below)
    gate, up = ref[:, :inter], ref[:, inter:]
    _close(out, gate * torch.sigmoid(gate) * up, 1e-5)
    assert (buf[m * inter:] == 77).all()


WIDE_ROUTES = [
    # M, N, K, whether gate/up with a workspace takes one round of wide tiles (they write no K parts) or 128-column tiles
    # whose last round is divided over K: on either side of the lines between the two
    (7, 37888, 3584, True), (128, 37888, 3584, True), (256, 37888, 3584, True), (24, 32896, 5120, True), (192, 32896, 3584, True),
    (96, 41088, 3584, True), (128, 41088, 3584, True), (256, 45056, 3584, True), (224, 32896, 1024, True), (7, 32896, 4096, True),
    (16, 41088, 8192, True), (56, 39424, 6144, True), (256, 41088, 2048, True), (128, 34816, 2048, True),
    (12, 37888, 3584, True), (90, 37888, 3584, True), (7, 41088, 3584, True), (20, 41088, 3584, True), (56, 45056, 3584, True),
    (150, 41088, 3584, True),      # with those above every build of either width
    (128, 32896, 3584, False), (97, 34816, 3584, False), (128, 37888, 8192, False), (193, 33664, 4096, False), (256, 34816, 5120, False),
    (224, 41088, 3584, False), (256, 43008, 5120, False), (7, 33664, 5120, False), (16, 41088, 6144, False), (56, 34816, 6144, False),
    (40, 53504, 4096, False), (160, 53504, 8192, False),
]


@pytest.mark.parametrize("m,n,k,wide", WIDE_ROUTES)
def test_gate_up_takes_wide_tiles_where_they_are_ahead(m, n, k, wide):
    from paper_2604_14889_amd import binding as M
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the rule was measured on 256 compute units")
    gen, a, w, ref = _inputs(m, n, k, m + n + k)
    blocks = ref.view(m, n // 64, 2, 32)          # gate and up rows interleaved in blocks of 32
    gate, up = blocks[:, :, 0].reshape(m, n // 2), blocks[:, :, 1].reshape(m, n // 2)
    want = gate * torch.sigmoid(gate) * up
    need = M.ms_gemm_workspace_bytes(m, n, k, 1)
    assert need > 0
    # too small a workspace and one off its alignment are none: nothing is written there
    buf = torch.empty(need + 16, dtype=torch.uint8, device="cuda")
    for ws, parts in ((buf[:need], not wide), (buf[:64], False), (buf[8:8 + need], False), (None, False)):
        buf.fill_(255)
        act = torch.full((m, n // 2), float("nan"), dtype=torch.bfloat16, device="cuda")
        M.ms_gemm_swiglu_bf16(a, w, act, ws)
        assert bool((buf != 255).any()) == parts
        _close(act, want, 2e-5 * (gate.abs() + 1) * (up.abs() + 1))


@pytest.mark.parametrize("m", [1, 12, 24, 90, 150, 256])
@pytest.mark.parametrize("inter", [16384 + 64, 20480 + 64])      # 160- and 192-column tiles, the last one partly past N
def test_wide_tiles_repeat_their_bits_on_either_alignment(m, inter):
    """16-byte pieces of a row where the destination allows it, 8-byte ones otherwise: the same bits, call after call, and
    nothing around the destination."""
    from paper_2604_14889_amd import binding as M
    k = 256
    gen, a, w, ref = _inputs(m, 2 * inter, k, m + inter)
    blocks = ref.view(m, inter // 32, 2, 32)
    gate, up = blocks[:, :, 0].reshape(m, inter), blocks[:, :, 1].reshape(m, inter)
    first = None
    for shift in (4, 8, 12, 8):
        buf = torch.full((m * inter + 16,), 77.0, dtype=torch.bfloat16, device="cuda")
        out = buf[shift:shift + m * inter].view(m, inter)
        assert out.data_ptr() % 16 == 2 * shift % 16
        M.ms_gemm_swiglu_bf16(a, w, out)
        _close(out, gate * torch.sigmoid(gate) * up, 2e-5 * (gate.abs() + 1) * (up.abs() + 1))
        assert (buf[:shift] == 77).all() and (buf[shift + m * inter:] == 77).all()
        first = out.clone() if first is None else first
        assert torch.equal(out.view(torch.int16), first.view(torch.int16))
