"""What a user of this library has it do, as cases that can be timed and compared.

The kinds of work, all through the calls of include/cassandra.h as paper_2605_26558_amd.binding
gives them:

  linear   one linear layer on its own: the draft product (speculation data only, 1 to 4 columns)
           or the verification product (exact weights, 1 to 32 columns), on raw, shared-exponent
           or unary-coded weights
  round    the passes of one speculative round of a Llama-3-shaped decoder over a filled cache:
           k draft passes, one verification pass over k + 1 columns, commit of the accepted
           positions; k = 0 is plain decoding.  One sequence, or up to four at once.
  prefill  a prompt through the target path into an empty cache, then the first token's logits
  append   the online encoder on a run of new K/V vectors
  encode   offline formatting of one weight matrix

Values are seeded stand-ins with the structure the method is made for: weights normal with
0.5 % of the input columns x20, log-normal activation norms, keys with four outlier channels per
head x10.  The token ids fed to the passes are given, not chained, so that a near tie between two
logits does not turn into another sequence of inputs.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2605_26558_amd import binding as B

SHAPES = {  # hidden, query heads, kv heads, feed-forward, vocabulary
    "8b": (4096, 32, 8, 14336, 128256),
    "70b": (8192, 64, 8, 28672, 128256),
    "tiny": (256, 4, 2, 512, 1000),
}


def _model(shape, **kw):
    hidden, n_q, n_kv, ffn, vocab = SHAPES[shape]
    c = {"hidden": hidden, "n_q": n_q, "n_kv": n_kv, "ffn": ffn, "vocab": vocab, "keep": 600, "trunc": 4,
         "form": "raw", "kv_form": "raw"}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest unit of work: one 4096 x 4096 layer at 25 % kept, one column of the draft pass
        {"name": "linear_draft_4096", "kind": "linear", "dir": "draft", "rows": 4096, "cols": 4096, "keep": 250,
         "trunc": 4, "ncols": 1, "form": "raw"},
        # the same layer in the verification of four drafts
        {"name": "linear_verify_4096", "kind": "linear", "dir": "verify", "rows": 4096, "cols": 4096, "keep": 250,
         "trunc": 4, "ncols": 5, "form": "raw"},
        # a layer whose sides divide by nothing, verified for several sequences at once
        {"name": "linear_verify_ragged", "kind": "linear", "dir": "verify", "rows": 11003, "cols": 5001, "keep": 700,
         "trunc": 3, "ncols": 20, "form": "raw"},
        # a small model at the start of a conversation: launches and latency, hardly any bytes
        {"name": "round_tiny", "kind": "round", **_model("tiny"), "layers": 2, "seqs": 1, "context": 203, "k": 4,
         "accept": 2},
        # the headline workload: the whole 8B-shaped model, batch 1, 8K of context, draft length 6
        {"name": "round_8b", "kind": "round", **_model("8b"), "layers": 32, "seqs": 1, "context": 8192, "k": 6,
         "accept": 4},
        # long contexts of four sequences of unequal length (traffic of the cache), draft length 4
        {"name": "round_8b_batch4", "kind": "round", **_model("8b"), "layers": 8, "seqs": 4, "context": 32768, "k": 4,
         "accept": 2},
        # wide layers: the 70B shape, draft length 8
        {"name": "round_70b", "kind": "round", **_model("70b"), "layers": 4, "seqs": 1, "context": 8192, "k": 8,
         "accept": 5},
        # the lossy configuration: shared exponents in weights and cache
        {"name": "round_8b_shared", "kind": "round", **_model("8b", form="shared", kv_form="shared"), "layers": 8,
         "seqs": 1, "context": 8192, "k": 6, "accept": 4},
        # the lossless small configuration: unary-coded exponents in the weights
        {"name": "round_8b_unary", "kind": "round", **_model("8b", form="unary"), "layers": 4, "seqs": 1,
         "context": 4096, "k": 4, "accept": 3},
        # a prompt of about 512 tokens before the first decode step
        {"name": "prefill_8b", "kind": "prefill", **_model("8b"), "layers": 4, "seqs": 1, "tokens": 509},
        # a prompt's K/V of one layer going into the cache, starting inside a page
        {"name": "append_1021", "kind": "append", "n_kv": 8, "tokens": 1021, "pos0": 37, "keep": 600, "trunc": 4,
         "kv_form": "raw"},
        # formatting the largest matrix of an 8B layer when a model is loaded
        {"name": "encode_28672x4096", "kind": "encode", "rows": 28672, "cols": 4096, "keep": 600, "trunc": 4,
         "act": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    keep, trunc = rng.choice([250, 400, 500, 600, 600, 600, 700, rng.randint(200, 1000)]), rng.choice([4, 4, 4, 0, 1, 2, 3, 5])
    kind = rng.choice(["linear", "linear", "linear", "round", "round", "round", "prefill", "append", "encode"])
    if kind in ("linear", "encode"):
        rows, cols = _log(rng, 256, 32768), _log(rng, 256, 16384)
        if rng.random() < 0.6:  # most layers are multiples of 64, some divide by nothing
            rows, cols = (rows + 63) // 64 * 64, (cols + 63) // 64 * 64
        rows = min(rows, 120_000_000 // cols)
        if kind == "encode":
            return {"kind": kind, "rows": rows, "cols": cols, "keep": keep, "trunc": trunc, "act": rng.random() < 0.7}
        form = rng.choice(["raw", "raw", "raw", "shared", "unary"])
        if form == "unary":  # its kernel holds x and the exponents of eight rows in LDS
            keep, cols = min(keep, 700), min(cols, 14336)
        which = rng.choice(["draft", "verify"])
        ncols = _log(rng, 1, 32) if which == "verify" else (rng.choice([1, 1, 2, 3, 4]) if form == "raw" else 1)
        return {"kind": kind, "dir": which, "rows": rows, "cols": cols, "keep": keep, "trunc": trunc, "ncols": ncols,
                "form": form}
    kv_form = rng.choice(["raw", "raw", "raw", "shared"])
    if kind == "append":
        return {"kind": kind, "n_kv": rng.choice([2, 4, 8]), "tokens": _log(rng, 1, 4096), "pos0": rng.randint(0, 500),
                "keep": keep, "trunc": trunc, "kv_form": kv_form}
    shape = rng.choice(["tiny", "8b", "8b", "70b", "other"])
    c = _model("8b" if shape == "other" else shape, keep=keep, trunc=trunc, kv_form=kv_form,
               form=rng.choice(["raw", "raw", "raw", "raw", "shared", "unary"]))
    if shape == "other":
        grp, n_kv = rng.choice([1, 2, 4, 7, 8]), rng.choice([2, 4, 8])
        c.update(n_q=grp * n_kv, n_kv=n_kv, hidden=8 * rng.randint(64, 800), ffn=8 * rng.randint(128, 2000),
                 vocab=_log(rng, 2000, 128256))
    if c["form"] == "unary":
        c["keep"] = min(keep, 700)
        c["form"] = "raw" if max(c["ffn"], c["hidden"]) > 14336 else "unary"
    layers = rng.randint(1, 4) if shape in ("8b", "tiny") else rng.randint(1, 2)
    if kind == "prefill":
        return {"kind": kind, **c, "layers": min(layers, 2), "seqs": 1, "tokens": _log(rng, 16, 512)}
    seqs, k = rng.choice([1, 1, 1, 2, 4]), rng.choice([0, 1, 2, 4, 6, 8])
    if shape == "70b" or c["form"] == "unary":  # a draft pass holds the columns' feed-forward values in LDS
        seqs = min(seqs, 2)
    k = min(k, 80 // (c["n_q"] // c["n_kv"]) - 1)
    return {"kind": kind, **c, "layers": layers, "seqs": seqs, "context": _log(rng, 64, 32768), "k": k,
            "accept": rng.randint(0, k)}


# Sizes of a model's weights.  The projections that add to the residual stream are 1 / sqrt(2 * 32)
# as large as the others, the usual scaling for a stack of 32 layers.  With 0.02 for all of them,
# random layers amplify a rounding of their input to 4 % of the logits of 32 layers (1.4 % with
# these), which would hide a wrong result.
_SIGMA = {"wqkv": 0.01, "wo": 0.01 / 8, "wgu": 0.01, "wd": 0.01 / 8}


# ---- inputs -----------------------------------------------------------------------------------

def _bits(t):
    return t.to(torch.bfloat16).view(torch.int16)


def _randn(gen, *shape):
    return torch.randn(shape, device="cuda", generator=gen)


def _weight(gen, rows, cols, sigma=0.02):
    w = _randn(gen, rows, cols).mul_(sigma)
    n_out = round(0.005 * cols)
    if n_out:
        w[:, torch.randperm(cols, device="cuda", generator=gen)[:n_out]] *= 20.0
    return _bits(w)


def _act_norm(gen, cols):
    return torch.exp(0.5 * _randn(gen, cols))


def _encoded(ctx, gen, rows, cols, case, sigma=0.02):
    return B.cas_encode_weight(ctx, _weight(gen, rows, cols, sigma), case["keep"], case["trunc"], _act_norm(gen, cols))


def _exp_mode(case):
    return B.CAS_EXP_SHARED if case["kv_form"] == "shared" else B.CAS_EXP_RAW


def _kv_values(gen, tokens, heads, outliers):
    K = _randn(gen, tokens, heads, 128)
    K[:, :, outliers] *= 10.0
    return _bits(K).contiguous(), _bits(_randn(gen, tokens, heads, 128)).contiguous()


def _contexts(case):
    """Committed positions of every sequence: the longest first, the others shorter by odd amounts."""
    n = case["context"]
    return [n, max(1, n - 27), max(1, (n * 5) // 8), max(1, n // 8 + 1)][: case["seqs"]]


def _columns(case):
    """Columns a pass may carry: what one round brings, 32 at most; a prompt goes in chunks of 16."""
    return 16 if case["kind"] == "prefill" else min(32, max(1, case["seqs"] * (case["k"] + 1)))


def _prepare_model(case, gen):
    hidden, n_q, n_kv, ffn, vocab, layers = (case[n] for n in ("hidden", "n_q", "n_kv", "ffn", "vocab", "layers"))
    prefill = case["kind"] == "prefill"
    lens = [0] if prefill else _contexts(case)
    max_pos = case["tokens"] + 8 if prefill else max(lens) + case["k"] + 8
    per_seq = 16 if prefill else case["k"] + 1
    pages = (max_pos + 63) // 64 + 1
    # partial results of the sequences that share an attention launch, one record per 64 positions
    partials = case["seqs"] * (pages * n_kv * per_seq * (n_q // n_kv) * 132 * 4 + 256)
    ctx = B.Context(workspace=torch.empty(max(64 << 20, partials), dtype=torch.uint8, device="cuda"))
    dims = (("wqkv", (n_q + 2 * n_kv) * 128, hidden), ("wo", hidden, n_q * 128), ("wgu", 2 * ffn, hidden),
            ("wd", hidden, ffn))
    gain = lambda: _bits(1.0 + 0.1 * _randn(gen, hidden))  # noqa: E731
    weights = []
    for _ in range(layers):
        layer = {n: _encoded(ctx, gen, r, c, case, _SIGMA[n]) for n, r, c in dims}
        layer["g_attn"], layer["g_ffn"] = gain(), gain()
        weights.append(layer)
    head = _encoded(ctx, gen, vocab, hidden, case)
    embed = _bits(_randn(gen, vocab, hidden))
    angle = torch.outer(torch.arange(max_pos, dtype=torch.float64),
                        500000.0 ** (-torch.arange(0, 128, 2, dtype=torch.float64) / 128))
    rope = torch.stack([angle.cos(), angle.sin()], -1).to(torch.float32).cuda().contiguous()
    shape = SimpleNamespace(hidden=hidden, n_layers=layers, n_q_heads=n_q, n_kv_heads=n_kv, head_dim=128, ffn=ffn,
                            vocab=vocab, rms_eps=1e-5)
    model = B.Model(ctx, shape, weights, head, embed, gain(), rope, max_cols=max(_columns(case), per_seq),
                    max_seqs=case["seqs"])
    if case["form"] != "raw":
        recode, use = (B.cas_mx_encode, model.use_mx) if case["form"] == "shared" else (B.cas_unary_encode, model.use_unary)
        for i, layer in enumerate(weights):
            for which, (n, _, _) in enumerate(dims):
                use(i, which, recode(ctx, layer[n]))
        use(-1, 0, recode(ctx, head))
    kv = B.KVCache(ctx, layers, n_kv, n_pages=pages * case["seqs"], max_seqs=case["seqs"], max_pages_per_seq=pages,
                   keep_permille=case["keep"], trunc_bits=case["trunc"], exp_mode=_exp_mode(case))
    for layer in range(layers):
        outliers = torch.randperm(128, device="cuda", generator=gen)[:4]
        for seq, n in enumerate(lens):
            if n:
                B.cas_kv_set_len(kv, seq, 0)
                B.cas_kv_append(ctx, kv, layer, seq, *_kv_values(gen, n, n_kv, outliers))
    for seq, n in enumerate(lens):
        B.cas_kv_set_len(kv, seq, n)
    s = SimpleNamespace(case=case, ctx=ctx, model=model, kv=kv, lens=lens)
    ids = lambda *sh: torch.randint(0, vocab, sh, device="cuda", generator=gen, dtype=torch.int32)  # noqa: E731
    if prefill:
        s.prompt, s.target, s.logits = ids(case["tokens"]), torch.empty(1, dtype=torch.int32, device="cuda"), \
            torch.empty((1, vocab), device="cuda")
        return s
    k, seqs = case["k"], case["seqs"]
    s.tokens = ids(seqs, k + 1)                      # pending token and drafts of every sequence
    s.steps = s.tokens.t().contiguous()              # the same, one row per draft pass
    s.drafted = torch.empty((max(k, 1), seqs), dtype=torch.int32, device="cuda")
    s.target = torch.empty(seqs * (k + 1), dtype=torch.int32, device="cuda")
    if seqs == 1:
        s.draft_logits = torch.empty((k, vocab), device="cuda")
        s.logits = torch.empty((k + 1, vocab), device="cuda")
    return s


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind in ("round", "prefill"):
        return _prepare_model(case, gen)
    ctx = B.Context(workspace=torch.empty(64 << 20, dtype=torch.uint8, device="cuda"))
    s = SimpleNamespace(case=case, ctx=ctx)
    if kind == "linear":
        s.w = _encoded(ctx, gen, case["rows"], case["cols"], case)
        if case["form"] != "raw":
            s.w = (B.cas_mx_encode if case["form"] == "shared" else B.cas_unary_encode)(ctx, s.w)
        s.x = _bits(_randn(gen, case["ncols"], case["cols"]))
        s.y = torch.empty((case["ncols"], case["rows"]), device="cuda")
    elif kind == "append":
        pages = (case["pos0"] + case["tokens"] + 63) // 64
        s.kv = B.KVCache(ctx, 1, case["n_kv"], n_pages=pages, max_seqs=1, max_pages_per_seq=pages,
                         keep_permille=case["keep"], trunc_bits=case["trunc"], exp_mode=_exp_mode(case))
        s.kv.spec_pool.zero_()
        s.kv.verif_pool.zero_()
        s.K, s.V = _kv_values(gen, case["tokens"], case["n_kv"], torch.randperm(128, device="cuda", generator=gen)[:4])
    else:
        s.W = _weight(gen, case["rows"], case["cols"])
        s.act = _act_norm(gen, case["cols"]) if case["act"] else None
    return s


# ---- one pass ---------------------------------------------------------------------------------

_LINEAR = {("draft", "raw"): B.cas_gemv_draft, ("draft", "shared"): B.cas_gemv_draft_mx,
           ("draft", "unary"): B.cas_gemv_draft_unary, ("verify", "raw"): B.cas_gemm_verify,
           ("verify", "shared"): B.cas_gemm_verify_mx, ("verify", "unary"): B.cas_gemm_verify_unary}


def _committed(s, layer, seq, n):
    K, V = B.cas_kv_read(s.ctx, s.kv, layer, seq, s.lens[seq], n, True)
    return [K.view(torch.bfloat16), V.view(torch.bfloat16)]


def _run_round(s):
    """The passes of a round on the given tokens, committed; the outputs are the logits (where one
    sequence is decoded) and the vectors that the last layer's cache received."""
    case, ctx, model, kv = s.case, s.ctx, s.model, s.kv
    k, seqs, n = case["k"], case["seqs"], case["accept"]
    last = case["layers"] - 1
    for seq in range(seqs):
        B.cas_kv_set_len(kv, seq, s.lens[seq])
    if seqs == 1:
        for i in range(k):
            B.cas_draft_step(ctx, model, kv, 0, s.tokens[0, i:], i, s.drafted[i], s.draft_logits[i])
        B.cas_verify_step(ctx, model, kv, 0, s.tokens, k, s.target, s.logits)
        B.cas_commit(ctx, model, kv, 0, n)
        return [s.draft_logits, s.logits, *_committed(s, last, 0, n + 1)]
    ids = list(range(seqs))
    for i in range(k):
        B.cas_draft_step_multi(ctx, model, kv, ids, [i] * seqs, s.steps[i], s.drafted[i])
    B.cas_verify_step_multi(ctx, model, kv, ids, [k] * seqs, s.tokens, s.target)
    out = []
    for seq in ids:
        B.cas_commit(ctx, model, kv, seq, n)
        out += _committed(s, last, seq, n + 1)
    return out


def run(s):
    case, kind = s.case, s.case["kind"]
    if kind == "linear":
        return _LINEAR[case["dir"], case["form"]](s.ctx, s.w, s.x, s.y)
    if kind == "round":
        return _run_round(s)
    if kind == "prefill":
        B.cas_kv_set_len(s.kv, 0, 0)
        B.cas_prefill(s.ctx, s.model, s.kv, 0, s.prompt[:-1])
        B.cas_verify_step(s.ctx, s.model, s.kv, 0, s.prompt[-1:], 0, s.target, s.logits)
        return s.logits
    if kind == "append":
        B.cas_kv_set_len(s.kv, 0, case["pos0"])
        B.cas_kv_append(s.ctx, s.kv, 0, 0, s.K, s.V)
        return [s.kv.spec_pool, s.kv.verif_pool]
    e = B.cas_encode_weight(s.ctx, s.W, case["keep"], case["trunc"], s.act)
    d = e.desc
    cut = lambda buf, off, words: buf[off: off + 4 * d.rows * words]  # noqa: E731  (a stream without its padding)
    return [cut(e.spec, d.off_bitmap, d.bw), cut(e.spec, d.off_spec, d.sw), cut(e.verif, d.off_lo, d.lw),
            cut(e.verif, d.off_pruned, d.pw)]


# ---- what a pass cannot do without ------------------------------------------------------------

def _row_bytes(cols, case, form, full):
    """Bytes of one selection group in the streams a pass reads (or the encoder writes)."""
    keep, t = case["keep"], case["trunc"]
    K = (keep * cols + 500) // 1000
    words = lambda bits: (bits + 31) // 32  # noqa: E731
    bw = words(cols)
    if form == "raw":
        spec = bw + words(K * (16 - t))
    elif form == "shared":
        spec = bw + (bw + 3) // 4 + words(K * (9 - t))
    else:  # sign and mantissa fields, and about 1.7 bits of exponent code per kept value
        spec = bw + words(K * (8 - t)) + words(int(1.7 * K))
    return 4 * (spec + (words(K * t) + words((cols - K) * 16) if full else 0))


def _matrix(rows, cols, ncols, case, full, form=None):
    """(bytes, flops) of one product with an encoded matrix."""
    kept = 1.0 if full else case["keep"] / 1000
    return (rows * _row_bytes(cols, case, form or case["form"], full) + ncols * (2 * cols + 4 * rows),
            2.0 * rows * cols * kept * ncols)


def _pass(case, ncols, lens, full, head=True):
    """(bytes, flops) of one pass of the model: `ncols` columns in all, shared evenly by the sequences."""
    hidden, n_q, n_kv, ffn, vocab = (case[n] for n in ("hidden", "n_q", "n_kv", "ffn", "vocab"))
    mats = [((n_q + 2 * n_kv) * 128, hidden), (hidden, n_q * 128), (2 * ffn, hidden), (hidden, ffn)] * case["layers"]
    got = [_matrix(r, c, ncols, case, full) for r, c in mats + ([(vocab, hidden)] if head else [])]
    per_pos = 2 * n_kv * _row_bytes(128, case, case["kv_form"], full)
    by = sum(g[0] for g in got) + case["layers"] * per_pos * sum(lens)
    fl = sum(g[1] for g in got) + case["layers"] * 4.0 * 128 * n_q * (ncols / len(lens)) * sum(lens)
    return by, fl


def work(case):
    kind = case["kind"]
    if kind == "linear":
        by, fl = _matrix(case["rows"], case["cols"], case["ncols"], case, case["dir"] == "verify")
    elif kind == "round":
        lens, k, seqs = _contexts(case), case["k"], case["seqs"]
        d, v = _pass(case, seqs, lens, False), _pass(case, seqs * (k + 1), lens, True)
        by, fl = k * d[0] + v[0], k * d[1] + v[1]
    elif kind == "prefill":
        # the weights once, the products of every position; the output head for the last one
        n = case["tokens"]
        by, fl = _pass(case, n, [n / 2], True, head=False)
        b2, f2 = _matrix(case["vocab"], case["hidden"], 1, case, True)
        by, fl = by + b2, fl + f2
    elif kind == "append":
        rows = 2 * case["n_kv"] * case["tokens"]
        by, fl = rows * (256 + _row_bytes(128, case, case["kv_form"], True)), 0.0
    else:
        by, fl = case["rows"] * (2 * case["cols"] + _row_bytes(case["cols"], case, "raw", True)), 0.0
    return {"bytes": float(by), "flops": float(fl)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("append", "encode"):
        return "exact"
    if kind == "linear":
        # sums of exact bf16 products in fp32: 2.3e-7 against float64 on the longest listed rows
        return {"rel": 2e-6, "max": 2e-5}
    # bf16 between the operations: another order of the sums moves roundings, and every layer adds to
    # the difference (1.4 % of the logits after 32 layers, against the same roundings around float64)
    return {"rel": min(0.03, 0.01 + 0.0025 * case["layers"])}
