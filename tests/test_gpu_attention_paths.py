"""The attention kernels' own edges against the oracle: row blocks, chunks, shares and the tails of
pages.  The tolerances are those of test_gpu_parity.py (fp32 1e-5 max-abs; bf16 2e-2 max-abs and 1e-2
mean-rel); pool bytes past a sequence's end are NaN throughout."""
import numpy as np
import pytest

import workloads as W
from tests.test_gpu_parity import check_out, oracle_attention, pids_for, run_gpu_attention, setup_pair, _mods

pytestmark = pytest.mark.gpu


def poison_tails(inp):
    """NaN into every slot past a sequence's end, in its last page and in the pages nobody owns."""
    sh = inp.shape
    nan = np.uint16(0x7FC0) if sh.dtype == "bf16" else np.float32(np.nan)
    owned = set()
    for n, pt in zip(sh.lengths, inp.page_tables):
        owned.update(pt)
        if n % W.PAGE_SIZE:
            inp.pool[:, pt[-1], :, :, n % W.PAGE_SIZE:, :] = nan
    for page in set(range(sh.n_pages)) - owned:
        inp.pool[:, page] = nan


def compare(sh, stream, ctx=None):
    M, _ = _mods()
    inp = W.attention_inputs(sh, 900, stream)
    poison_tails(inp)
    ses, ora, ids = setup_pair(inp)
    with ses:
        pos = pids_for(inp, M)
        got = run_gpu_attention(ses, inp, ids, pos, ctx_new=ctx)
        again = run_gpu_attention(ses, inp, ids, pos, ctx_new=ctx)
        want = oracle_attention(ora, inp, ids, pos, ctx_new=ctx)
        assert np.isfinite(got).all()
        check_out(got, want, sh.dtype, str(sh)[:200])
        return got, again


GENERAL = [
    # dtype, Hq, Hkv, D, n_verify, n_foresight, lengths: rows per KV head in blocks of 16, up to 4 (D = 64) or 2 (D = 128) per workgroup
    ("f32", 4, 4, 64, 16, 0, [0, 1, 15, 16, 17]),          # one full block
    ("bf16", 4, 4, 64, 17, 0, [63, 64, 65, 1000]),         # two blocks, one row in the second
    ("f32", 9, 3, 64, 4, 9, [48, 333]),                    # 39 rows: three blocks
    ("bf16", 16, 4, 64, 5, 4, [2000, 31]),                 # 36 rows, many shares and a short sequence beside a long one
    ("f32", 8, 2, 64, 16, 0, [129, 0]),                    # 64 rows: four full blocks
    ("bf16", 20, 4, 64, 13, 0, [100]),                     # 65 rows: two chunks
    ("bf16", 7, 1, 64, 64, 0, [16, 200]),                  # 448 rows, four in-flight tiles
    ("f32", 3, 3, 128, 5, 4, [255, 256, 257]),             # D = 128, one block
    ("f32", 8, 2, 128, 7, 0, [400, 15]),                   # 28 rows: two blocks
    ("f32", 8, 2, 128, 9, 0, [17]),                        # 36 rows: two chunks
    ("bf16", 65, 1, 128, 1, 1, [300, 0]),                  # more than 64 heads per KV head: bf16, D = 128
    ("bf16", 80, 1, 128, 0, 1, [33]),
]


@pytest.mark.parametrize("dtype,hq,hkv,d,nv,nf,lengths", GENERAL)
def test_general_kernel_row_blocks_chunks_and_page_tails(dtype, hq, hkv, d, nv, nf, lengths):
    sh = W.AttnShape("general", dtype, len(lengths), hq, hkv, d, nv, nf, lengths, 1.0 if dtype == "f32" else 0.5, 10000.0)
    got, again = compare(sh, hq * 100 + nv)
    assert (got == again).all()                            # the general kernel is reproducible bit for bit
    n_q = nv + nf
    ctx = np.asarray([[(i * 7 + b) % (n_q + 1) for i in range(n_q)] for b in range(len(lengths))], np.int32)
    compare(sh, hq * 100 + nv, ctx)


SPLIT = [
    # Hq, Hkv, n_verify, n_foresight, lengths: bf16, head_dim 128, calls of the share-per-workgroup kernel
    (28, 4, 4, 3, [0]),                                    # in-flight tile only
    (28, 4, 5, 4, [1, 31, 32, 33]),                        # a tile with one page, a full tile, one token in the second
    (28, 4, 1, 0, [16, 17, 48]),                           # a tile whose second page does not exist
    (32, 8, 5, 4, [4100]),
    (28, 4, 4, 3, [9000, 40]),                             # many shares, most of them empty for the second sequence
    (28, 4, 4, 3, [12000]),                                # more shares than one round trip of the second launch takes
    (16, 2, 8, 0, [700]),                                  # 64 rows
    (4, 4, 16, 0, [130]),                                  # one row block
    (28, 4, 10, 0, [65, 0]),                               # two chunks, the second with one query
    (28, 4, 33, 0, [100]),                                 # two in-flight tiles, the second with one token
    (28, 4, 64, 0, [1000, 15]),
    (64, 1, 3, 2, [100]),                                  # 64 heads per KV head: a chunk per query
    (48, 1, 64, 0, [40]),                                  # 64 chunks, unfilled rows in every one
]


@pytest.mark.parametrize("hq,hkv,nv,nf,lengths", SPLIT)
def test_share_per_workgroup_kernel_tiles_chunks_and_shares(hq, hkv, nv, nf, lengths):
    sh = W.AttnShape("split", "bf16", len(lengths), hq, hkv, 128, nv, nf, lengths, 0.5, 1000000.0)
    got, again = compare(sh, hq * 100 + nv)
    assert (got == again).all()
    n_q = nv + nf
    ctx = np.asarray([[(i * 7 + b) % (n_q + 1) for i in range(n_q)] for b in range(len(lengths))], np.int32)
    compare(sh, hq * 100 + nv, ctx)


def test_share_per_workgroup_kernel_follows_the_device_length_and_agrees_with_the_streaming_kernel():
    """Rows committed on the device after the host last looked belong to the last share; the same call
    forced onto the streaming kernel (fault injection with a generous bound) gives the same rows."""
    import torch
    M, S = _mods()
    sh = W.AttnShape("grow", "bf16", 2, 28, 4, 128, 5, 4, [60, 500], 0.5, 1000000.0, slack_pages=1.0)
    inp = W.attention_inputs(sh, 901)
    ses, ora, ids = setup_pair(inp)
    with ses:
        pos = pids_for(inp, M)
        q, kn, vn = (S.to_device(x, M.MS_BF16) for x in (inp.q, inp.k_new, inp.v_new))
        p = S.ints_dev(pos).view(sh.batch, sh.n_q)
        first = ses.attention(0, ids, 5, 4, q, kn, vn, p)
        acc = S.ints_dev([5, 3])
        for _ in range(4):
            M.ms_commit_accepted_device(ses.cache, ids, acc, sh.n_q, 5, kn, vn, p)
        lagging = ses.attention(0, ids, 5, 4, q, kn, vn, p)
        assert not torch.equal(first, lagging)
        M.ms_cache_sync(ses.cache)
        assert ses.lengths(ids) == [80, 512]
        caught_up = ses.attention(0, ids, 5, 4, q, kn, vn, p)
        M.ms_attention_fault_injection(ses.cache, 1 << 22, 0)
        streamed = ses.attention(0, ids, 5, 4, q, kn, vn, p)
        for other in (caught_up, streamed):
            check_out(S.to_host_f32(lagging), S.to_host_f32(other).astype(np.float64), "bf16", "after device-side commits")


NOT_FINITE = [
    # dtype, Hq, Hkv, D, n_verify, n_foresight, lengths: one and several shares, one and several chunks of rows
    ("f32", 8, 8, 64, 4, 3, [30]),
    ("f32", 8, 2, 128, 7, 2, [400, 15]),
    ("bf16", 16, 4, 64, 5, 4, [700, 31]),
    ("bf16", 7, 1, 64, 20, 0, [100]),
    ("bf16", 66, 1, 128, 1, 2, [300]),
    ("f32", 4, 4, 64, 64, 0, [16]),                        # two shares, in the second of which the first rows see nothing
]


@pytest.mark.parametrize("where", ["v_new", "cached_v", "cached_k"])
@pytest.mark.parametrize("dtype,hq,hkv,d,nv,nf,lengths", NOT_FINITE)
def test_general_kernel_keeps_infinities_where_they_belong(dtype, hq, hkv, d, nv, nf, lengths, where):
    """An infinite or NaN value of an in-flight token reaches the rows that see the token and no others; an
    infinite cached value its own column; a score of -infinity has no weight."""
    M, _ = _mods()
    sh = W.AttnShape("inf", dtype, len(lengths), hq, hkv, d, nv, nf, lengths, 1.0 if dtype == "f32" else 0.5, 10000.0)
    inp = W.attention_inputs(sh, 902, hq)
    inf, nan = (np.uint16(0x7F80), np.uint16(0x7FC0)) if dtype == "bf16" else (np.float32(np.inf), np.float32(np.nan))
    neg = np.uint16(0xFF80) if dtype == "bf16" else np.float32(-np.inf)
    if where == "v_new":
        inp.v_new[:, -1, :, 5] = inf                       # the last token: only its own rows see it
        inp.v_new[0, nv - 1, 0, 3] = nan
    else:
        page = inp.page_tables[0][0]
        inp.pool[0, page, :, 1 if where == "cached_v" else 0, 3, 7] = inf if where == "cached_v" else neg
    ses, ora, ids = setup_pair(inp)
    with ses:
        pos = pids_for(inp, M)
        got = run_gpu_attention(ses, inp, ids, pos).astype(np.float64)
        with np.errstate(invalid="ignore"):
            want = oracle_attention(ora, inp, ids, pos)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want))
    finite = np.isfinite(want)
    assert finite.sum() >= 0.3 * want.size and not finite.all()
    check_out(got, np.where(finite, want, np.nan), dtype, f"{where} {sh}"[:200])


ROUTES = [
    # Hq, Hkv, n_verify, n_foresight, lengths, kernel: one long sequence among short ones is levelled by the planned
    # kernels only; with lengths not that far apart, or few tiles, the share-per-workgroup kernel is ahead
    (28, 4, 5, 4, [12000] + 15 * [100], "pv_attn_mfma_stream"),
    (28, 4, 5, 4, [500 + 1071 * i for i in range(8)], "pv_attn_mfma_stream"),
    (32, 8, 5, 4, [8000] + 7 * [64], "pv_attn_mfma_stream"),
    (28, 4, 5, 4, [100 + 100 * i for i in range(16)], "pv_attn_mfma_split"),
    (28, 4, 4, 3, [16000, 100], "pv_attn_mfma_split"),
    (28, 4, 4, 3, [4096], "pv_attn_mfma_split"),
    (28, 4, 64, 0, [9000] + 7 * [64], "pv_attn_mfma_wide"),
    (32, 8, 41, 0, [6000] + 7 * [64], "pv_attn_mfma_wide"),
    (28, 4, 64, 0, [4000] + 7 * [64], "pv_attn_mfma_split"),
    (28, 4, 64, 0, [2000], "pv_attn_mfma_split"),
]


@pytest.mark.parametrize("hq,hkv,nv,nf,lengths,kernel", ROUTES)
def test_skewed_batches_run_on_the_kernel_that_levels_them(hq, hkv, nv, nf, lengths, kernel):
    import torch
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the rule was measured on 256 compute units")
    M, S = _mods()
    sh = W.AttnShape("skew", "bf16", len(lengths), hq, hkv, 128, nv, nf, lengths, 0.5, 1000000.0)
    inp = W.attention_inputs(sh, 903, len(lengths))
    ses, ora, ids = setup_pair(inp)
    with ses:
        pos = pids_for(inp, M)
        got = run_gpu_attention(ses, inp, ids, pos)
        assert M.ms_attention_last_kernel(ses.cache).split("+")[0] == kernel
        from oracle import memosight_oracle as O
        from tests.test_gpu_parity import as_f32
        for b in (0, len(lengths) - 1):                        # the longest and a short one (or the other way round)
            want = O.attention_rows(ora, 0, ids[b], as_f32(inp.q[b], "bf16"), as_f32(inp.k_new[b], "bf16"), as_f32(inp.v_new[b], "bf16"),
                                    pos[b], O.default_ctx_new(nv, nf), rows=[(i, h) for i in (0, nv + nf - 1) for h in range(0, hq, 3)])
            check_out(got[b], want, "bf16", f"sequence {b}")


@pytest.mark.parametrize("hq,hkv,nv,nf,lengths", [
    # one launch sums the split kernel's shares, by blocks of 32 x 32 outputs or by quarters of them: at most 8, 16 and 32
    # shares, more than one batch of them, one and two row blocks, on either side of the line between the two
    (28, 4, 4, 3, [200]), (28, 4, 4, 3, [460]), (28, 4, 4, 3, [3000]), (8, 2, 1, 3, [9000]), (28, 4, 5, 4, [33, 700]),
    (28, 4, 5, 4, [33, 700, 1]), (16, 8, 9, 0, [500]), (16, 8, 9, 0, [500, 64]), (28, 4, 41, 0, [130]),
    (8, 2, 1, 3, [11000]),                                 # 345 tiles in 39 shares (9000 tokens are 32: one batch)
])
def test_shares_are_summed_by_blocks_and_by_quarters(hq, hkv, nv, nf, lengths):
    sh = W.AttnShape("fold", "bf16", len(lengths), hq, hkv, 128, nv, nf, lengths, 0.5, 1000000.0)
    got, again = compare(sh, 950 + len(lengths))
    assert np.array_equal(got, again)


@pytest.mark.parametrize("dtype,hq,hkv,d,nv,lengths", [
    # rows of the second launch of the general kernel: one, a workgroup of one wave full and one row more, as many rows as
    # workgroups of one wave take (131072 elements on 256 compute units) and 31 rows more
    ("f32", 1, 1, 64, 1, [200]), ("f32", 4, 4, 64, 1, [130]), ("f32", 5, 5, 64, 1, [130]), ("f32", 3, 3, 128, 1, [300]),
    ("bf16", 32, 8, 64, 64, [40]), ("bf16", 33, 11, 64, 63, [40]),
])
def test_partials_of_the_general_kernel_are_summed_by_one_or_four_waves(dtype, hq, hkv, d, nv, lengths):
    compare(W.AttnShape("combine", dtype, len(lengths), hq, hkv, d, nv, 0, lengths, 1.0 if dtype == "f32" else 0.5, 10000.0), 970 + hq)
