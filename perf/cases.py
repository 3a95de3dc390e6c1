"""The work a program has this library do, as cases that can be timed and compared.

Four kinds of case, each a pass through the public entry points (binding.py, session.py, decoder.py):

  attention  every layer's Predict+Verify attention of one step over the paged cache: the decode
             step (a few queries), a prompt chunk or memory-token pass (up to 64 queries), and the
             other caches the entry point takes (fp32, head_dim 64)
  block      the kernels of one decoder block around the attention: embedding rows, norm, fused
             Q/K/V, output projection + norm, gate/up + SwiGLU, down projection + norm
  step       Decoder.step: embedding, all blocks, final norm, LM head, greedy token
  cache      a reasoning step's life in the cache: import, accept + commit for every speculative
             step, compaction of the segment into memory tokens, release

Sizes: Qwen2.5-7B's widths (28 / 4 heads of 128, hidden 3584, MLP 18944, vocabulary 152064), the
32 / 8 head layout of Llama-3.1-8B (hidden 4096, MLP 14336), 8 / 8 heads of 64 for fp32 caches, and
generic ones.  Everything is drawn on the GPU from the seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2604_14889_amd import binding as M
from paper_2604_14889_amd.decoder import Decoder, DecoderConfig, DecoderTensors, LayerTensors
from paper_2604_14889_amd.session import Session

PAGE = 16
EPS = 1e-6
DEV = "cuda:0"

QWEN = {"hidden": 3584, "inter": 18944, "heads_q": 28, "heads_kv": 4, "dim": 128}
LLAMA = {"hidden": 4096, "inter": 14336, "heads_q": 32, "heads_kv": 8, "dim": 128}


def _attention(name, dtype="bf16", dim=128, heads_q=28, heads_kv=4, batch=1, kv_lo=4096, kv_hi=4096, verify=4, foresight=3,
               layers=28):
    case = {"kind": "attention", "dtype": dtype, "dim": dim, "heads_q": heads_q, "heads_kv": heads_kv, "batch": batch,
            "kv_lo": kv_lo, "kv_hi": kv_hi, "verify": verify, "foresight": foresight, "layers": layers}
    return dict(case, name=name) if name else case


def listed():
    return [
        # one user, the attention of a whole step (all 28 layers): launch latency and the fixed part of a launch
        _attention("attn_b1_kv4k"),
        # the headline decode point: 32 sequences of 8192 cached tokens, 5 verify + 4 foresight queries
        _attention("attn_b32_kv8k", batch=32, kv_lo=8192, kv_hi=8192, verify=5, foresight=4, layers=2),
        # the same batch as a server sees it: lengths all over 1k .. 16k, no length a multiple of a tile
        _attention("attn_b32_ragged", batch=32, kv_lo=1021, kv_hi=16383, verify=5, foresight=4, layers=2),
        # a prompt enters in chunks of 64 causal queries; the memory-token pass looks the same
        _attention("attn_chunk64_kv2k", kv_lo=2000, kv_hi=2000, verify=64, foresight=0),
        # small models have heads of 64
        _attention("attn_d64_b16_kv4k", dim=64, heads_q=16, heads_kv=4, batch=16, kv_lo=4000, kv_hi=4096, verify=5, foresight=4,
                   layers=4),
        # fp32 cache (accuracy work, reference runs): 8 heads of 64
        _attention("attn_f32_b4_kv1k", dtype="f32", dim=64, heads_q=8, heads_kv=8, batch=4, kv_lo=320, kv_hi=1500, layers=4),
        # a block's projections for one sequence of 4 + 3 queries, eight sequences, sixty-four sequences
        dict(QWEN, kind="block", rows=7, name="block_rows7"),
        dict(QWEN, kind="block", rows=56, name="block_rows56"),
        dict(QWEN, kind="block", rows=448, name="block_rows448"),
        # the model's whole step with the LM head, one sequence and a batch (fewer layers than the model has)
        dict(QWEN, kind="step", vocab=152064, batch=1, kv=8000, verify=4, foresight=3, layers=4, name="step_b1"),
        dict(QWEN, kind="step", vocab=152064, batch=32, kv=2000, verify=4, foresight=3, layers=2, name="step_b32"),
        # sixteen reasoning steps in the cache: 14 speculative steps each, then compaction at ratio 7
        {"kind": "cache", "heads_kv": 4, "dim": 128, "layers": 28, "batch": 16, "kv": 250, "steps": 14, "verify": 5, "foresight": 4,
         "ratio": 7, "name": "cache_b16"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _attention_fit(case, most_bytes):
    """As many layers (up to 28) and as long a cache as keep a pass within most_bytes of cache."""
    esize = 4 if case["dtype"] == "f32" else 2
    row = 2 * case["heads_kv"] * case["dim"] * esize
    per_layer = case["batch"] * (case["kv_lo"] + case["kv_hi"]) / 2 * row
    if per_layer > most_bytes:
        scale = most_bytes / per_layer
        case["kv_lo"], case["kv_hi"] = max(1, int(case["kv_lo"] * scale)), max(1, int(case["kv_hi"] * scale))
        per_layer = most_bytes
    case["layers"] = max(1, min(28, int(most_bytes / per_layer)))
    return case


def draw(rng):
    pick = rng.random()
    if pick < 0.35:     # decode attention
        heads_q, heads_kv = rng.choice([(28, 4), (28, 4), (32, 8)])
        lo = _log_int(rng, 100, 16000)
        hi = lo if rng.random() < 0.4 else min(16383, lo * rng.randint(2, 16))
        verify, foresight = rng.choice([(1, 3), (4, 3), (5, 4), (5, 0), (2, 5)])
        return _attention_fit(_attention(None, heads_q=heads_q, heads_kv=heads_kv, batch=_log_int(rng, 1, 64), kv_lo=lo, kv_hi=hi,
                                         verify=verify, foresight=foresight), 8e8)
    if pick < 0.47:     # wide steps: prompt chunks, memory-token passes, per-position foresight
        heads_q, heads_kv = rng.choice([(28, 4), (32, 8)])
        lo = _log_int(rng, 64, 6000)
        return _attention_fit(_attention(None, heads_q=heads_q, heads_kv=heads_kv, batch=_log_int(rng, 1, 8), kv_lo=lo, kv_hi=lo,
                                         verify=rng.randint(17, 64), foresight=0), 1e8)
    if pick < 0.60:     # the other caches
        dtype, dim, heads_q, heads_kv = rng.choice([("bf16", 64, 16, 4), ("bf16", 64, 8, 8), ("f32", 64, 8, 8), ("f32", 128, 16, 4)])
        lo = _log_int(rng, 50, 3000)
        verify, foresight = rng.choice([(4, 3), (5, 4), (1, 3)])
        return _attention_fit(_attention(None, dtype=dtype, dim=dim, heads_q=heads_q, heads_kv=heads_kv, batch=_log_int(rng, 1, 12),
                                         kv_lo=lo, kv_hi=min(4000, int(lo * rng.uniform(1, 4))), verify=verify, foresight=foresight), 3e7)
    if pick < 0.85:
        return dict(rng.choice([QWEN, QWEN, LLAMA]), kind="block", rows=_log_int(rng, 2, 448))
    if pick < 0.93:
        return dict(QWEN, kind="step", vocab=152064, batch=_log_int(rng, 1, 32), kv=_log_int(rng, 200, 2000), verify=4, foresight=3,
                    layers=rng.randint(1, 2))
    return {"kind": "cache", "heads_kv": 4, "dim": 128, "layers": rng.choice([8, 28]), "batch": _log_int(rng, 1, 16),
            "kv": rng.randint(20, 260), "steps": rng.randint(4, 14), "verify": 5, "foresight": 4, "ratio": rng.choice([4, 7])}


# ---- inputs ------------------------------------------------------------------------------------------

class State:
    """What a program holds between calls; gives the cache handle back."""

    def __init__(self, **kw):
        self.__dict__.update(kw)

    def __del__(self):
        ses = self.__dict__.get("ses")
        if ses is not None:
            ses.close()


def _generator(seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    return gen


def _normal(gen, *shape, sigma=1.0, dtype=torch.bfloat16):
    return torch.empty(*shape, dtype=dtype, device=DEV).normal_(0.0, sigma, generator=gen)


def _lengths(case, seed):
    """Cache lengths spread evenly over kv_lo .. kv_hi, in an order of the seed's."""
    lo, hi, n = case["kv_lo"], case["kv_hi"], case["batch"]
    out = [lo + (hi - lo) * i // max(1, n - 1) for i in range(n)] if n > 1 else [hi]
    random.Random(seed).shuffle(out)
    return out


def _pages_of(n_tokens):
    return -(-n_tokens // PAGE)


def _page_tables(lengths, seed):
    """Disjoint page lists out of a pool with a tenth to spare, in random order."""
    n_pages = int(sum(_pages_of(n) for n in lengths) * 1.1) + 2 * len(lengths)
    perm, out, at = np.random.RandomState(seed % (1 << 31)).permutation(n_pages), [], 0
    for n in lengths:
        out.append(perm[at:at + _pages_of(n)].astype(np.int32))
        at += _pages_of(n)
    return n_pages, out


def _step_inputs(case, seed, n_layers, lengths):
    n_pages, tables = _page_tables(lengths, seed)
    dt = M.MS_F32 if case.get("dtype") == "f32" else M.MS_BF16
    ses = Session(n_layers, case["heads_q"], case["heads_kv"], case["dim"], n_pages, dt, 1000000.0, max_seqs=len(lengths),
                  max_pages_per_seq=max(len(t) for t in tables) + 8)
    gen = _generator(seed)
    ses.pool.normal_(0.0, 1.0, generator=gen)
    ids = [M.ms_seq_import(ses.cache, n, t) for n, t in zip(lengths, tables)]
    first = np.asarray([3 * n + 1 for n in lengths], np.int32)   # a compressed cache holds about a third of the tokens
    pos = torch.from_numpy(M.ms_step_positions(first, case["verify"], case["foresight"])).to(DEV)
    return ses, gen, tables, M.int_array(ids), pos


def _prepare_attention(case, seed):
    lengths = _lengths(case, seed)
    ses, gen, tables, ids, pos = _step_inputs(case, seed, case["layers"], lengths)
    n_q = case["verify"] + case["foresight"]
    dt = ses.tdtype
    q = _normal(gen, case["layers"], case["batch"], n_q, case["heads_q"], case["dim"], sigma=2.0, dtype=dt)
    k = _normal(gen, case["layers"], case["batch"], n_q, case["heads_kv"], case["dim"], dtype=dt)
    v = _normal(gen, case["layers"], case["batch"], n_q, case["heads_kv"], case["dim"], dtype=dt)
    layers = [(li, q[li], k[li], v[li]) for li in range(case["layers"])]
    out = torch.empty_like(q)
    return State(kind="attention", ses=ses, ids=ids, pos=pos, layers=layers, q=q, k=k, v=v, out=out, outs=list(out), tables=tables,
                 lengths=lengths, verify=case["verify"], foresight=case["foresight"])


def _run_attention(s):
    for (li, q, k, v), out in zip(s.layers, s.outs):
        s.ses.attention(li, s.ids, s.verify, s.foresight, q, k, v, s.pos, out=out)
    return s.out


def _layer_weights(case, gen):
    hid, inter = case["hidden"], case["inter"]
    qd, kd = case["heads_q"] * case["dim"], case["heads_kv"] * case["dim"]

    def norm():
        return (1.0 + 0.1 * torch.randn(hid, device=DEV, generator=gen)).to(torch.bfloat16)

    return {"ln1": norm(), "wq": _normal(gen, qd, hid, sigma=hid ** -0.5), "bq": _normal(gen, qd, sigma=0.1),
            "wk": _normal(gen, kd, hid, sigma=hid ** -0.5), "bk": _normal(gen, kd, sigma=0.1),
            "wv": _normal(gen, kd, hid, sigma=hid ** -0.5), "bv": _normal(gen, kd, sigma=0.1),
            "wo": _normal(gen, hid, qd, sigma=qd ** -0.5), "ln2": norm(),
            "w_gate_up": _normal(gen, 2 * inter, hid, sigma=hid ** -0.5), "w_down": _normal(gen, hid, inter, sigma=inter ** -0.5)}


def _split(k, want):
    steps = k // 32
    return max(s for s in range(1, want + 1) if steps % s == 0 and (s == 1 or steps // s >= 4))


def _block_inputs(case, seed):
    gen = _generator(seed)
    raw = _layer_weights(case, gen)
    rows, hid = case["rows"], case["hidden"]
    table = _normal(gen, 512, hid)
    tokens = torch.randint(0, 512, (rows,), device=DEV, generator=gen, dtype=torch.int32)
    attn = _normal(gen, rows, case["heads_q"] * case["dim"], sigma=0.5)
    ln3 = (1.0 + 0.1 * torch.randn(hid, device=DEV, generator=gen)).to(torch.bfloat16)
    return raw, table, tokens, attn, ln3


def _prepare_block(case, seed):
    raw, table, tokens, attn, ln3 = _block_inputs(case, seed)
    rows, hid, inter = case["rows"], case["hidden"], case["inter"]
    qd, kd = case["heads_q"] * case["dim"], case["heads_kv"] * case["dim"]
    lw = LayerTensors(*(raw[n] for n in ("ln1", "wq", "bq", "wk", "bk", "wv", "bv", "wo", "ln2", "w_gate_up", "w_down")))
    # K divided as Decoder divides it for a step of that many rows
    few = rows <= 256
    sq, so, sd = (_split(hid, 7 if few else 4), max(2, _split(qd, 8 if few else 7)), max(2, _split(inter, 16 if few else 8)))
    need = max(M.ms_gemm_workspace_bytes(rows, qd + 2 * kd, hid, sq), M.ms_gemm_add_rmsnorm_workspace_bytes(rows, hid, qd, so),
               M.ms_gemm_workspace_bytes(rows, 2 * inter, hid, 1), M.ms_gemm_add_rmsnorm_workspace_bytes(rows, hid, inter, sd), 16)

    def buf(*shape, dtype=torch.bfloat16):
        return torch.empty(*shape, dtype=dtype, device=DEV)

    return State(kind="block", w=lw, table=table, tokens=tokens, attn=attn, ln3=ln3, splits=(sq, so, sd),
                 ws=buf(need, dtype=torch.uint8), h=buf(rows, hid, dtype=torch.float32), x1=buf(rows, hid), q=buf(rows, qd), k=buf(rows, kd),
                 v=buf(rows, kd), x2=buf(rows, hid), act=buf(rows, inter), x3=buf(rows, hid))


def _run_block(s):
    w = s.w
    sq, so, sd = s.splits
    M.ms_embed_rows(s.table, s.tokens, s.h)
    M.ms_add_rmsnorm(s.h, None, w.ln1, EPS, s.x1)
    M.ms_gemm_bf16(s.x1, w.wqkv, w.bqkv, [s.q, s.k, s.v], sq, s.ws)
    M.ms_gemm_add_rmsnorm_bf16(s.attn, w.wo, s.h, w.ln2, EPS, s.x2, so, s.ws)
    M.ms_gemm_swiglu_bf16(s.x2, w.w_gate_up_blocked, s.act, s.ws)
    M.ms_gemm_add_rmsnorm_bf16(s.act, w.w_down, s.h, s.ln3, EPS, s.x3, sd, s.ws)
    return {"x1": s.x1, "q": s.q, "k": s.k, "v": s.v, "x2": s.x2, "act": s.act, "h": s.h, "x3": s.x3}


def _step_weights(case, gen):
    layers = [_layer_weights(case, gen) for _ in range(case["layers"])]
    embed = _normal(gen, case["vocab"], case["hidden"])
    norm = (1.0 + 0.1 * torch.randn(case["hidden"], device=DEV, generator=gen)).to(torch.bfloat16)
    lm_head = _normal(gen, case["vocab"], case["hidden"], sigma=case["hidden"] ** -0.5)
    return layers, embed, norm, lm_head


def _step_tokens(case, gen):
    return torch.randint(0, case["vocab"], (case["batch"], case["verify"] + case["foresight"]), device=DEV, generator=gen, dtype=torch.int32)


def _prepare_step(case, seed):
    lengths = [case["kv"]] * case["batch"]
    ses, gen, tables, ids, pos = _step_inputs(case, seed, case["layers"], lengths)
    raw, embed, norm, lm_head = _step_weights(case, gen)
    tokens = _step_tokens(case, gen)
    layers = [LayerTensors(*(r[n] for n in ("ln1", "wq", "bq", "wk", "bk", "wv", "bv", "wo", "ln2", "w_gate_up", "w_down"))) for r in raw]
    cfg = DecoderConfig(case["layers"], case["hidden"], case["inter"], case["vocab"], case["heads_q"], case["heads_kv"], case["dim"], EPS)
    dec = Decoder(cfg, DecoderTensors(embed, layers, norm, lm_head), ses, case["batch"] * (case["verify"] + case["foresight"]))
    return State(kind="step", ses=ses, dec=dec, ids=ids, pos=pos, tokens=tokens, verify=case["verify"], foresight=case["foresight"])


def _run_step(s):
    logits, _ = s.dec.step(s.ids, s.tokens, s.pos, s.verify, s.foresight)
    k, v = s.dec.step_kv()
    return {"logits": logits, "k": k, "v": v}


def _accepts(case):
    """Drafts accepted per speculative step and sequence: the same for every seed, so that the work is."""
    rng = random.Random(case["batch"] * 10007 + case["kv"])
    return [[rng.choice([1, 2, 3, 4, 4, 5]) for _ in range(case["batch"])] for _ in range(case["steps"])]


def _cache_inputs(case, seed):
    B, L, n_q = case["batch"], case["layers"], case["verify"] + case["foresight"]
    acc = _accepts(case)
    grown = [sum(a[b] for a in acc) for b in range(B)]
    n_mem = [M.ms_ama_count(g, case["ratio"]) for g in grown]
    per = _pages_of(case["kv"])
    n_pages = B * (per + _pages_of(max(grown)) + 2)
    first = [3 * case["kv"] + 1 + b for b in range(B)]
    mem_pos = [p for b in range(B) for p in M.ms_upl_positions(first[b], grown[b], case["ratio"])]
    rng = np.random.RandomState(seed % (1 << 31))
    draft = rng.randint(0, 150000, size=(case["steps"], B, case["verify"])).astype(np.int32)
    target = draft.copy()
    for s, row in enumerate(acc):
        for b, a in enumerate(row):
            target[s, b, a:] = draft[s, b, a:] + 1
    gen = _generator(seed)
    k = _normal(gen, L, B, n_q, case["heads_kv"], case["dim"])
    v = _normal(gen, L, B, n_q, case["heads_kv"], case["dim"])
    mk = _normal(gen, L, sum(n_mem), case["heads_kv"], case["dim"])
    mv = _normal(gen, L, sum(n_mem), case["heads_kv"], case["dim"])
    return gen, acc, grown, n_mem, per, n_pages, first, mem_pos, draft, target, k, v, mk, mv


def _prepare_cache(case, seed):
    B = case["batch"]
    gen, acc, grown, n_mem, per, n_pages, first, mem_pos, draft, target, k, v, mk, mv = _cache_inputs(case, seed)
    ses = Session(case["layers"], 7 * case["heads_kv"], case["heads_kv"], case["dim"], n_pages, M.MS_BF16, 1000000.0, max_seqs=B,
                  max_pages_per_seq=n_pages)
    ses.pool.normal_(0.0, 1.0, generator=gen)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(np.asarray(x, np.int32))).to(DEV)  # noqa: E731
    n_q = case["verify"] + case["foresight"]
    return State(kind="cache", ses=ses, case=dict(case), tables=[np.arange(b * per, (b + 1) * per, dtype=np.int32) for b in range(B)],
                 n_mem=n_mem, first0=dev(first), first=dev(first), mem_pos=dev(mem_pos), draft=list(dev(draft)), target=list(dev(target)),
                 k=k, v=v, mk=mk, mv=mv, pos=torch.zeros(B, n_q, dtype=torch.int32, device=DEV),
                 acc=torch.zeros(case["steps"], B, dtype=torch.int32, device=DEV), nxt=torch.zeros(case["steps"], B, dtype=torch.int32, device=DEV))


def _run_cache(s):
    c, cache = s.case, s.ses.cache
    B, nv, nf = c["batch"], c["verify"], c["foresight"]
    ids = M.int_array([M.ms_seq_import(cache, c["kv"], t) for t in s.tables])
    s.first.copy_(s.first0)
    for i in range(c["steps"]):
        M.ms_step_positions_device(s.first, nv, nf, s.pos)
        M.ms_accept(B, nv, s.draft[i], s.target[i], None, s.acc[i], s.nxt[i])
        M.ms_commit_accepted_device(cache, ids, s.acc[i], nv + nf, nv, s.k, s.v, s.pos, s.first)
    grown = [M.ms_seq_len(cache, b) - c["kv"] for b in ids]
    M.ms_compact_segment(cache, ids, [c["kv"]] * B, grown, s.n_mem, s.mk, s.mv, s.mem_pos)
    for b in ids:
        M.ms_seq_free(cache, b)
    return {"pool": s.ses.pool, "accept_len": s.acc, "next_token": s.nxt, "first_pid": s.first}


_PREPARE = {"attention": _prepare_attention, "block": _prepare_block, "step": _prepare_step, "cache": _prepare_cache}
_RUN = {"attention": _run_attention, "block": _run_block, "step": _run_step, "cache": _run_cache}


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


def run(state):
    return _RUN[state.kind](state)


# ---- what a pass cannot do without --------------------------------------------------------------------

def _attention_work(case, lengths, esize):
    n_q = case["verify"] + case["foresight"]
    row = case["heads_kv"] * case["dim"] * esize
    tokens = sum(lengths)
    b = 2 * tokens * row + 4 * sum(_pages_of(n) for n in lengths)
    b += case["batch"] * n_q * (2 * case["heads_q"] * case["dim"] * esize + 2 * row)
    f = 4.0 * case["heads_q"] * case["dim"] * n_q * (tokens + case["batch"] * n_q / 2)
    return b, f


def _block_work(case, rows):
    hid, inter = case["hidden"], case["inter"]
    qd, kd = case["heads_q"] * case["dim"], case["heads_kv"] * case["dim"]
    params = hid * (qd + 2 * kd) + qd * hid + 3 * hid * inter
    acts = rows * (2 * hid + 2 * hid + 2 * (qd + 2 * kd) + 2 * qd + 4 * hid + 2 * hid + 2 * inter + 2 * hid)
    return 2 * params + acts, 2.0 * rows * params


def work(case):
    if case["kind"] == "attention":
        b, f = _attention_work(case, _lengths(case, 0), 4 if case["dtype"] == "f32" else 2)
        return {"bytes": case["layers"] * b, "flops": case["layers"] * f}
    if case["kind"] == "block":
        b, f = _block_work(case, case["rows"])
        return {"bytes": b, "flops": f}
    if case["kind"] == "step":
        rows = case["batch"] * (case["verify"] + case["foresight"])
        hid, kd = case["hidden"], case["heads_kv"] * case["dim"]
        weights = case["layers"] * (hid * (case["heads_q"] * case["dim"] + 2 * kd) + case["heads_q"] * case["dim"] * hid + 3 * hid * case["inter"])
        head = case["vocab"] * hid
        kv = case["layers"] * 2 * case["batch"] * case["kv"] * kd * 2
        _, f = _attention_work(case, [case["kv"]] * case["batch"], 2)
        return {"bytes": 2 * (weights + head) + kv + rows * (2 * hid + 2 * case["vocab"]) + case["layers"] * rows * 4 * kd,
                "flops": 2.0 * rows * (weights + head) + case["layers"] * f}
    acc = _accepts(case)
    rows = sum(sum(a) for a in acc) + sum(M.ms_ama_count(sum(a[b] for a in acc), case["ratio"]) for b in range(case["batch"]))
    row = case["layers"] * 2 * case["heads_kv"] * case["dim"] * 2
    return {"bytes": 2 * rows * row, "flops": 6.0 * rows * case["layers"] * case["heads_kv"] * case["dim"]}


def tolerance(case):
    # about four times the distance to the 64-bit results: 4e-7 (fp32 attention; up to 1e-6 for longer caches), 4e-3 (bf16
    # attention: rotated rows, probabilities and results are rounded to 8 bits), 4e-4 (cache: rotated keys are rounded once,
    # everything else is copied), 3e-3 (a block), 5e-3 (logits after a few layers; the same inputs twice differ by as much)
    if case["kind"] == "attention":
        return {"rel": 5e-6} if case["dtype"] == "f32" else {"rel": 1e-2}
    return {"rel": {"cache": 2e-3, "block": 1e-2, "step": 2e-2}[case["kind"]]}


# ---- the same in 64 bits --------------------------------------------------------------------------------

def _rotate(x, pos, base=1000000.0):
    """x [..., rows, heads, dim] in fp64, pos [rows]; pairs (i, i + dim/2), the angle rounded to fp32 as the library defines it."""
    half = x.shape[-1] // 2
    inv = torch.from_numpy((base ** (-2.0 * np.arange(half) / x.shape[-1])).astype(np.float32)).to(x.device)
    angle = (pos.to(torch.float32)[:, None] * inv[None, :]).double()
    cos, sin = torch.cos(angle)[:, None, :], torch.sin(angle)[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], dim=-1)


def _attend(pool_layer, table, n, q, k_new, v_new, pos, verify):
    """One sequence and layer: q [n_q, Hq, D], k_new / v_new [n_q, Hkv, D], all fp64."""
    n_q, hq, dim = q.shape
    hkv = k_new.shape[1]
    group = hq // hkv
    pages = pool_layer[torch.from_numpy(table.astype(np.int64)).to(pool_layer.device)].double()      # [pages, Hkv, 2, 16, D]
    kv = pages.permute(2, 1, 0, 3, 4).reshape(2, hkv, -1, dim)[:, :, :n]
    keys = torch.cat([kv[0], _rotate(k_new, pos).transpose(0, 1)], dim=1)        # [Hkv, n + n_q, D]
    vals = torch.cat([kv[1], v_new.transpose(0, 1)], dim=1)
    qr = _rotate(q, pos).transpose(0, 1).reshape(hkv, group * n_q, dim)          # rows: head in group, query
    i = torch.arange(n_q, device=q.device)
    seen = (i[None, :] < torch.clamp(i, max=verify)[:, None]) | (i[None, :] == i[:, None])
    s = torch.matmul(qr, keys.transpose(1, 2).contiguous()) * dim ** -0.5
    s[:, :, n:].masked_fill_(~seen.repeat(group, 1)[None], float("-inf"))
    o = torch.matmul(torch.softmax(s, dim=-1), vals)
    return o.reshape(hkv * group, n_q, dim).transpose(0, 1)


def _exact_attention(case, seed):
    s = _prepare_attention(case, seed)
    out = torch.empty(s.q.shape, dtype=torch.float64, device=DEV)
    for li in range(case["layers"]):
        for b in range(case["batch"]):
            out[li, b] = _attend(s.ses.pool[li], s.tables[b], s.lengths[b], s.q[li, b].double(), s.k[li, b].double(), s.v[li, b].double(),
                                 s.pos[b], case["verify"])
    return out


def _rms(h, w):
    return h / torch.sqrt((h * h).mean(dim=-1, keepdim=True) + EPS) * w.double()


def _linear(x, w, bias=None):
    y = torch.matmul(x, w.double().t().contiguous())
    return y if bias is None else y + bias.double()


def _mlp(x, r):
    inter = r["w_gate_up"].shape[0] // 2
    gate, up = _linear(x, r["w_gate_up"][:inter]), _linear(x, r["w_gate_up"][inter:])
    return gate * torch.sigmoid(gate) * up


def _exact_block(case, seed):
    r, table, tokens, attn, ln3 = _block_inputs(case, seed)
    h = table[tokens.long()].double()
    x1 = _rms(h, r["ln1"])
    h = h + _linear(attn.double(), r["wo"])
    x2 = _rms(h, r["ln2"])
    act = _mlp(x2, r)
    h = h + _linear(act, r["w_down"])
    return {"x1": x1, "q": _linear(x1, r["wq"], r["bq"]), "k": _linear(x1, r["wk"], r["bk"]), "v": _linear(x1, r["wv"], r["bv"]), "x2": x2,
            "act": act, "h": h, "x3": _rms(h, ln3)}


def _exact_step(case, seed):
    lengths = [case["kv"]] * case["batch"]
    ses, gen, tables, ids, pos = _step_inputs(case, seed, case["layers"], lengths)
    raw, embed, norm, lm_head = _step_weights(case, gen)
    tokens = _step_tokens(case, gen)
    B, n_q, hq, hkv, dim = case["batch"], case["verify"] + case["foresight"], case["heads_q"], case["heads_kv"], case["dim"]
    h = embed[tokens.reshape(-1).long()].double()
    ks, vs = [], []
    for li, r in enumerate(raw):
        x = _rms(h, r["ln1"])
        q, k, v = (_linear(x, r["w" + n], r["b" + n]) for n in "qkv")
        ks.append(k.view(B * n_q, hkv, dim))
        vs.append(v.view(B * n_q, hkv, dim))
        attn = torch.cat([_attend(ses.pool[li], tables[b], lengths[b], q.view(B, n_q, hq, dim)[b], ks[-1].view(B, n_q, hkv, dim)[b],
                                  vs[-1].view(B, n_q, hkv, dim)[b], pos[b], case["verify"]).reshape(n_q, hq * dim) for b in range(B)])
        h = h + _linear(attn, r["wo"])
        h = h + _linear(_mlp(_rms(h, r["ln2"]), r), r["w_down"])
    logits = _linear(_rms(h, norm), lm_head)
    ses.close()
    return {"logits": logits, "k": torch.stack(ks), "v": torch.stack(vs)}


def _exact_cache(case, seed):
    gen, acc, grown, n_mem, per, n_pages, first, mem_pos, draft, target, k, v, mk, mv = _cache_inputs(case, seed)
    L, B, hkv, dim, kv = case["layers"], case["batch"], case["heads_kv"], case["dim"], case["kv"]
    pool = _normal(gen, L, n_pages, hkv, 2, PAGE, dim).double()      # drawn as prepare() draws it
    tables = [list(range(b * per, (b + 1) * per)) for b in range(B)]
    length, pid = [kv] * B, list(first)
    free = list(range(B * per, n_pages))                             # ascending; the lowest free page is taken

    def store(b, key, value, p):                                     # key, value [L, Hkv, D]
        if length[b] % PAGE == 0:
            tables[b].append(free.pop(0))
        page, slot = tables[b][length[b] // PAGE], length[b] % PAGE
        pool[:, page, :, 0, slot] = _rotate(key.double()[:, None], torch.tensor([p], device=DEV))[:, 0]
        pool[:, page, :, 1, slot] = value.double()
        length[b] += 1

    for row in acc:
        for b, a in enumerate(row):
            for j in range(a):
                store(b, k[:, b, j], v[:, b, j], pid[b] + j)
            pid[b] += a
    at = 0
    for b in range(B):
        keep = _pages_of(kv)
        free = sorted(free + tables[b][keep:])
        del tables[b][keep:]
        length[b] = kv
        for j in range(n_mem[b]):
            store(b, mk[:, at + j], mv[:, at + j], mem_pos[at + j])
        at += n_mem[b]
    return {"pool": pool, "accept_len": None, "next_token": None, "first_pid": None}


_EXACT = {"attention": _exact_attention, "block": _exact_block, "step": _exact_step, "cache": _exact_cache}


def exact(case, seed):
    return _EXACT[case["kind"]](case, seed)
