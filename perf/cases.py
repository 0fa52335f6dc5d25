"""The work that a user of the verifier has it do, as cases that can be timed and compared.

A case names a call of the public entry points (`session.VerifierSession`, `binding`) and its sizes:

  verify   one verifier pass over `seqs` sequences x `window` inputs with the logits of every row, followed by the
           accept rule (`verify` + `commit`: the inner step of the decode - verify - rollback loop)
  decode   one step of the fast path (`llm42_decode_step`), which produces the candidates
  prefill  the deterministic prefill of `seqs` prompts in passes of `chunk` rows per sequence

The models are the repository's two shapes with random bf16 weights N(0, 0.02^2) (one set per shape, made once per
process: a serving program holds one model for all of its calls); cached K and V are seeded noise and token ids random, as
in bench.py.  The lengths of a case follow from the case alone, so that every seed of it costs the same.
"""
import math

import numpy as np
import torch

from paper_2601_17768_amd import binding as B
from paper_2601_17768_amd import workloads as wl
from paper_2601_17768_amd.session import VerifierSession

SHAPES = {"8b": wl.LLAMA_8B, "tiny": wl.TINY}
MAX_POSITION = 16384
MAX_CACHED_TOKENS = 590_000       # of a drawn case; the largest listed one caches about as many
KV_RETURNED_BELOW = 3_000_000_000  # values: larger caches are not handed out as a result (a copy would not fit beside them)


def listed():
    return [
        # A two-layer model and a handful of rows: nothing but launches and latency.  The repository's small test shape,
        # for programs that check the protocol or speculate with a small model.
        dict(name="verify_tiny_4x8", do="verify", model="tiny", seqs=4, window=8, lengths="fixed:100"),
        # The candidate loop of a single interactive request: one token, every weight read once.
        dict(name="decode_1", do="decode", model="8b", seqs=1, lengths="fixed:512"),
        # The same loop for a group of ordinary size at chat-like lengths (the group of the loop statistics).
        dict(name="decode_24", do="decode", model="8b", seqs=24, lengths="sharegpt"),
        # Verification of a single request, window 32 behind a 512-token prompt: the smallest configuration of bench.py.
        dict(name="verify_1x32", do="verify", model="8b", seqs=1, window=32, lengths="fixed:512"),
        # A small group with odd sizes near the ends of its requests: windows only partly filled.
        dict(name="verify_5x13_ragged", do="verify", model="8b", seqs=5, window=13, lengths="sharegpt", ragged=True),
        # Grouped verification at its cheapest, 256 rows a pass, chat-like lengths.
        dict(name="verify_8x32", do="verify", model="8b", seqs=8, window=32, lengths="sharegpt"),
        # A large group with a small window over long documents: attention weighs as much as the weights.
        dict(name="verify_32x16_long", do="verify", model="8b", seqs=32, window=16, lengths="arxiv"),
        # Sampled requests (temperature above zero) of odd number and window, partly filled.
        dict(name="verify_27x37_sampled", do="verify", model="8b", seqs=27, window=37, lengths="sharegpt", ragged=True,
             temperature=0.7),
        # The 32-sequence configuration of bench.py: 2048 rows, lengths log-normal.
        dict(name="verify_32x64", do="verify", model="8b", seqs=32, window=64, lengths="lognormal"),
        # The 128-sequence configuration of bench.py, its headline: 4096 rows, contexts 1024 - 8192, 77 GB of K and V.
        dict(name="verify_128x32", do="verify", model="8b", seqs=128, window=32, lengths="uniform:1024:8192"),
        # A single prompt of ordinary, odd length.
        dict(name="prefill_1x700", do="prefill", model="8b", seqs=1, chunk=256, lengths="fixed:700"),
        # A batch of long prompts, 4096 rows a pass.
        dict(name="prefill_8x2048", do="prefill", model="8b", seqs=8, chunk=512, lengths="fixed:2048"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    kind = rng.choice(["verify", "verify", "verify", "verify", "decode", "decode", "prefill", "prefill", "tiny"])
    if kind == "tiny":
        return dict(do="verify", model="tiny", seqs=_log_int(rng, 1, 32), window=_log_int(rng, 2, 32),
                    lengths="fixed:%d" % _log_int(rng, 16, 600), ragged=rng.random() < 0.5)
    if kind == "prefill":
        seqs = _log_int(rng, 1, 8)
        return dict(do="prefill", model="8b", seqs=seqs, chunk=_log_int(rng, 32, 512),
                    lengths=rng.choice(["fixed:%d" % _log_int(rng, 40, 2048), "uniform:%d:%d" % (32, _log_int(rng, 64, 2048))]))
    lengths = rng.choice(["sharegpt", "lognormal", "arxiv", "fixed:%d" % _log_int(rng, 30, 8000),
                          "uniform:%d:%d" % (_log_int(rng, 16, 1024), _log_int(rng, 1200, 8192))])
    longest = {"sharegpt": 2000, "lognormal": 2000, "arxiv": 9000}.get(lengths) or int(lengths.split(":")[-1])
    seqs = _log_int(rng, 1, min(128, MAX_CACHED_TOKENS // longest))
    if kind == "decode":
        case = dict(do="decode", model="8b", seqs=seqs, lengths=lengths)
    else:
        window = _log_int(rng, 4, min(512, 4096 // seqs))
        case = dict(do="verify", model="8b", seqs=seqs, window=window, lengths=lengths, ragged=rng.random() < 0.5)
    if rng.random() < 0.25:
        case["temperature"] = rng.choice([0.6, 0.7, 1.0])
    return case


# ---- lengths -------------------------------------------------------------------------------------------------------
def _lengths(case):
    """(cached tokens, input rows) per sequence; for prefill (0, prompt length)."""
    n, kind = case["seqs"], case["lengths"]
    room = case.get("window", 1)
    rng = wl.rng_for(7, n, room)
    head, _, rest = kind.partition(":")
    if head == "fixed":
        ctx = np.full(n, int(rest), dtype=np.int64)
    elif head == "uniform":
        lo, hi = (int(x) for x in rest.split(":"))
        ctx = wl.uniform_lengths(rng, n, lo, hi)
    elif head == "lognormal":      # the lengths of bench.py's 32-sequence configuration
        ctx = wl.lognormal_lengths(rng, n, 6.0, 1.0, 16, 4096) + wl.lognormal_lengths(rng, n, 5.3, 0.9, 1, 2048)
    else:                          # dataset-shaped: a prompt and a uniformly drawn point of the output (sweep.py)
        from paper_2601_17768_amd.sweep import contexts_for
        ctx = np.minimum(contexts_for(head, rng, n, room, MAX_POSITION), 16000)
    ctx = ctx.astype(np.int32)
    if case["do"] == "prefill":
        return np.zeros(n, dtype=np.int32), ctx
    rows = rng.integers(1, room + 1, size=n).astype(np.int32) if case.get("ragged") else np.full(n, room, dtype=np.int32)
    return ctx, rows


# ---- models --------------------------------------------------------------------------------------------------------
_sessions = {}


def _session(name):
    if name not in _sessions:
        shape, gen = SHAPES[name], torch.Generator(device="cuda").manual_seed(42)

        def matrix(*dims):
            return torch.empty(dims, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=gen)

        d, f, hd = shape.d_model, shape.d_ffn, shape.head_dim
        gain = torch.ones(d, dtype=torch.bfloat16, device="cuda")
        layers = [dict(attn_norm=gain, wq=matrix(shape.n_q_heads * hd, d), wk=matrix(shape.n_kv_heads * hd, d),
                       wv=matrix(shape.n_kv_heads * hd, d), wo=matrix(d, shape.n_q_heads * hd), ffn_norm=gain,
                       w_gate=matrix(f, d), w_up=matrix(f, d), w_down=matrix(d, f)) for _ in range(shape.n_layers)]
        weights = dict(embed=matrix(shape.vocab, d), final_norm=gain, lm_head=matrix(shape.vocab, d), layers=layers)
        _sessions[name] = VerifierSession(shape, weights, max_position=MAX_POSITION)
        del weights, layers
        torch.cuda.empty_cache()
    return _sessions[name]


# ---- one case ------------------------------------------------------------------------------------------------------
def prepare(case, seed):
    sess = _session(case["model"])
    shape, n = sess.shape, case["seqs"]
    ctx, rows = _lengths(case)
    rng = wl.rng_for(seed, 11)
    table, blocks = wl.make_block_table(rng, ctx + (rows if case["do"] == "prefill" else case.get("window", 1)), 16, spare_blocks=4)
    state = dict(do=case["do"], sess=sess, table=torch.as_tensor(table, device="cuda"), sampling=None)
    if case.get("temperature"):
        state["request_ids"] = torch.as_tensor(rng.integers(0, 1 << 40, size=n), device="cuda")
        state["sampling"] = B.make_sampling(case["temperature"], seed, state["request_ids"])
    if case["do"] == "prefill":
        state["kv"] = sess.kv_cache(blocks)
        state["prompts"] = [wl.random_tokens(rng, int(m), shape.vocab) for m in rows]
        state["chunk"] = case["chunk"]
        return state
    kv = torch.empty((shape.n_layers, 2, blocks, shape.n_kv_heads, 16 * shape.head_dim), dtype=torch.bfloat16, device="cuda")
    state["kv"] = kv.normal_(generator=torch.Generator(device="cuda").manual_seed(seed))
    state["lens"] = torch.as_tensor(ctx, device="cuda")
    window = case.get("window", 1)
    state["max_context"] = int(ctx.max()) + window
    ids = torch.as_tensor(wl.random_tokens(rng, n * window, shape.vocab).reshape(n, window), device="cuda")
    if case["do"] == "decode":
        state["tokens"] = ids.view(n)
        state["next"] = torch.empty(n, dtype=torch.int32, device="cuda")
        state["status"] = torch.empty(n, dtype=torch.int32, device="cuda")
        state["workspace"] = sess.workspace(n, 1, state["max_context"])
        return state
    state["candidates"] = ids
    state["n_valid"] = torch.as_tensor(rows, device="cuda") if case.get("ragged") else None
    state["all"] = torch.arange(n, dtype=torch.int32, device="cuda")
    state["logits"] = torch.zeros((n, window, shape.vocab), dtype=torch.float32, device="cuda")
    return state


def run(state):
    sess, kv, table = state["sess"], state["kv"], state["table"]
    out = {}
    if state["do"] == "prefill":
        out["first"] = sess.prefill(kv, table, state["prompts"], window=state["chunk"], sampling=state["sampling"])
    elif state["do"] == "decode":
        B.llm42_decode_step(sess.model, kv, kv.shape[2], table, state["lens"], state["tokens"], state["max_context"],
                            state["next"], state["workspace"], state["status"], sampling=state["sampling"])
        out.update(next=state["next"], status=state["status"])
    else:
        lens = state["lens"].clone()          # the commit advances it; the state keeps its own
        tokens, status, logits = sess.verify(kv, table, lens, state["candidates"], state["n_valid"], dump_seq_ids=state["all"],
                                             max_context=state["max_context"], out_logits=state["logits"],
                                             sampling=state["sampling"])
        counts, committed, rolled = sess.commit(state["candidates"], tokens, lens, state["n_valid"])
        out.update(tokens=tokens, status=status, logits=logits, counts=counts, committed=committed, rolled=rolled, lens=lens)
    if kv.numel() <= KV_RETURNED_BELOW:
        out["kv"] = kv
    return out


def work(case):
    """Every weight matrix, cached key and value, and token's embedding read once, every new key and value and logit written
    once; two operations per weight and row, four per query feature, row and key."""
    shape = SHAPES[case["model"]]
    ctx, rows = (x.astype(np.float64) for x in _lengths(case))
    total = rows.sum()
    lm = shape.d_model * shape.vocab
    logit_rows = case["seqs"] if case["do"] == "prefill" else total
    keys = (rows * ctx + rows * (rows + 1) / 2).sum()
    nbytes = shape.gemm_params * 2 + (ctx + rows).sum() * shape.kv_bytes_per_token + total * shape.d_model * 2
    if case["do"] == "verify":
        nbytes += total * shape.vocab * 4
    flops = 2.0 * (shape.gemm_params - lm) * total + 2.0 * lm * logit_rows
    flops += 4.0 * keys * shape.n_layers * shape.n_q_heads * shape.head_dim
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    # The library's contract: every reduction runs under a fixed, documented schedule (llm42_schedule_info), so a token
    # and a logit are the same bits in any batch and from one build to the next.  A looser check would not hold either:
    # with random weights the two best logits of a row lie close together.  Measured: the sums of the two residual
    # projections in another order move the 32-layer model's logits by 1.5 % (2-norm) and change one token in 28.
    return "exact"
