"""The projections' tiles of 256 columns (wide outputs, up to 256 rows): row blocks, K ranges shorter than the pipeline, a last
tile of 128 columns, the divided last round with and without room for its parts, each epilogue.  Against the fp64 product;
one bf16 rounding (2^-8 with a safety factor) plus the fp32 accumulation error."""
import pytest
import torch

from tests.test_gpu_gemm_rows import _close, _inputs

pytestmark = pytest.mark.gpu

ROWS = [129, 160, 161, 192, 193, 224, 225, 256]


@pytest.mark.parametrize("m", ROWS)
def test_wide_outputs_by_rows_and_steps(m):
    from paper_2604_14889_amd import binding as M
    # 257 tiles of 256 and half a one: a last round of two tiles; K steps of 32: two, fewer than the stages, more
    for n, k in ((65536, 64), (65536 + 256 + 128, 128), (65536 + 128, 320), (131072 + 128, 192), (65536 + 384, 1024)):
        gen, a, w, ref = _inputs(m, n, k, m * 11 + k)
        bias = torch.empty(n, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
        need = M.ms_gemm_workspace_bytes(m, n, k, 1)
        for ws in (torch.full((max(need, 16),), 255, dtype=torch.uint8, device="cuda"), None):
            outs = [torch.full((m, c), float("nan"), dtype=torch.bfloat16, device="cuda") for c in (384, n - 384)]
            M.ms_gemm_bf16(a, w, bias, outs, 1, ws)
            assert M.ms_gemm_last_kernel() == "gemm_cols_bf16"
            _close(torch.cat(outs, dim=1), ref + bias.double())
            again = [torch.empty_like(o) for o in outs]
            M.ms_gemm_bf16(a, w, bias, again, 1, ws)
            assert all(torch.equal(x, y) for x, y in zip(outs, again))


@pytest.mark.parametrize("m", [129, 200, 256])
def test_gate_up_and_greedy_token_on_wide_tiles(m):
    from paper_2604_14889_amd import binding as M
    for inter, k in ((32768, 192), (32768 + 64, 640)):
        gen, a, w, ref = _inputs(m, 2 * inter, k, m * 13 + k)
        b = ref.view(m, inter // 32, 2, 32)
        gate, up = b[:, :, 0].reshape(m, inter), b[:, :, 1].reshape(m, inter)
        want = gate * torch.sigmoid(gate) * up
        need = M.ms_gemm_workspace_bytes(m, 2 * inter, k, 1)
        for ws in (torch.full((max(need, 16),), 255, dtype=torch.uint8, device="cuda"), None):
            out = torch.full((m, inter), float("nan"), dtype=torch.bfloat16, device="cuda")
            M.ms_gemm_swiglu_bf16(a, w, out, ws)
            assert M.ms_gemm_last_kernel() == "gemm_cols_bf16"
            # the factors' fp32 errors (1e-6 of the largest) times the other factor
            _close(out, want, 1e-5 * float(gate.abs().max() * up.abs().max()))
        n = 2 * inter
        tok = torch.full((m,), -1, dtype=torch.int32, device="cuda")
        keys = torch.empty(M.ms_lm_head_argmax_workspace_bytes(m, n, k), dtype=torch.uint8, device="cuda")
        M.ms_lm_head_argmax_bf16(a, w, tok, keys)
        best = ref.max(dim=1).values
        got = ref.gather(1, tok.long()[:, None])[:, 0]
        assert float((best - got).max()) <= 1e-5 * float(ref.abs().max())
