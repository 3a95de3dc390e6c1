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
