"""The streaming and the wide attention kernel at the parity tests' shapes, most of which the
share-per-workgroup kernel takes by itself: the same tests with that kernel left out (the fault injection's
switch, with the default bound and healthy counters), and a look at which kernel ran."""
import pytest

from tests import test_gpu_full_size as F
from tests import test_gpu_parity as P

pytestmark = pytest.mark.gpu

STREAM, WIDE = "pv_attn_mfma_stream", "pv_attn_mfma_wide"
DEFAULT_POLLS = 1 << 22


@pytest.fixture
def planned(monkeypatch):
    """Every Session from here on runs the planned kernels; yields the set of kernels its attention calls ran."""
    M, S = P._mods()
    ran = set()
    init, attention = S.Session.__init__, S.Session.attention

    def init_planned(self, *a, **kw):
        init(self, *a, **kw)
        M.ms_attention_fault_injection(self.cache, DEFAULT_POLLS, 0)

    def attention_noted(self, *a, **kw):
        out = attention(self, *a, **kw)
        ran.add(M.ms_attention_last_kernel(self.cache))
        return out

    monkeypatch.setattr(S.Session, "__init__", init_planned)
    monkeypatch.setattr(S.Session, "attention", attention_noted)
    return ran


def expected(hq, hkv, n_q):
    return STREAM if n_q <= 16 and n_q * (hq // hkv) <= 64 else WIDE


@pytest.mark.parametrize("dtype,hq,hkv,d,nv,nf,lengths", [s for s in P.SMALL if s[0] == "bf16" and s[3] == 128])
def test_small_shapes(planned, dtype, hq, hkv, d, nv, nf, lengths):
    P.test_attention_small_shapes_match_oracle(dtype, hq, hkv, d, nv, nf, lengths)
    assert planned == {expected(hq, hkv, nv + nf)}


@pytest.mark.parametrize("case", range(16))
def test_random_batches_of_boundary_lengths(planned, case):
    """Empty sequences, segments that end exactly on a tile, shares that cross several sequences."""
    P.test_attention_random_batches_of_boundary_lengths(case)
    assert len(planned) == 1 and planned <= {STREAM, WIDE}


def test_repeated_launches_with_many_partials_per_pair(planned):
    """The race check of the streaming kernel's closing: up to 25 partials per pair, whichever share ends last folds them."""
    P.test_repeated_launches_agree_with_many_partials_per_pair()
    assert planned == {STREAM}


def test_layer_pool_above_4_gib(planned):
    """The builds with 64-bit page bases, fixed and first-come tile assignment."""
    P.test_layer_pool_above_4_gib()
    assert planned == {STREAM}


def test_wide_step_after_device_side_commits(planned):
    P.test_wide_step_after_device_side_commits()
    assert planned == {WIDE}


def test_per_position_foresight_layout(planned):
    P.test_per_position_foresight_layout_wide_step()
    assert WIDE in planned


def test_foresight_rows_are_independent(planned):
    P.test_gpu_foresight_rows_independent_and_page_permutation_invariant()
    assert planned == {STREAM}


@pytest.mark.parametrize("nv,nf,lengths,scale,kernel", [(5, 4, [3000, 70, 0, 517], 0.2, STREAM), (41, 0, [700], 0.03, WIDE)])
def test_a_scale_of_the_callers(planned, nv, nf, lengths, scale, kernel):
    F.test_attention_with_a_scale_of_the_callers("bf16", 28, 4, 128, nv, nf, lengths, scale)
    assert planned == {kernel}
