"""Logits and new K / V of a sequence are the same bits at every row count of a pass, at the 8B model's layer
widths (one layer): the row counts below lie on both sides of every line at which a kernel changes its tile or its
rows per workgroup.  The reference is the sequence verified alone, which test_gpu_mid.py holds to the oracle; the
reduction schedule is part of the interface, so the comparison is exact."""
import numpy as np
import pytest
import torch

from helpers import wl
from gpu_helpers import VerifierSession, gpu_kv_tokens
from paper_2601_17768_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
WINDOW, CONTEXT = 16, 40


@pytest.fixture(scope="module")
def env():
    shape = wl.LLAMA_8B.replace(n_layers=1, vocab=4096)
    sess = VerifierSession(shape, wl.make_weights(shape, seed=47), max_position=128, device=DEV)
    yield shape, sess
    sess.close()


def _run(shape, sess, n_seq, slot, n_valid=None, bad_token_of=None, expect_status=None):
    rng = wl.rng_for(47, 3)
    kv_target = torch.empty((2, 4, shape.n_kv_heads, 16 * shape.head_dim), dtype=torch.bfloat16, device=DEV)
    kv_target.normal_(generator=torch.Generator(device=DEV).manual_seed(1))
    target = wl.random_tokens(rng, WINDOW, shape.vocab)
    rng = wl.rng_for(47, 4, n_seq)
    lens = rng.integers(1, 70, size=n_seq).astype(np.int32)
    lens[slot] = CONTEXT
    table, blocks = wl.make_block_table(rng, lens + WINDOW, 16, spare_blocks=2)
    bt = torch.as_tensor(table, device=DEV)
    kv = sess.kv_cache(blocks)
    kv.normal_(generator=torch.Generator(device=DEV).manual_seed(n_seq))
    kv[0][:, bt[slot, :4].long()] = kv_target
    cand = wl.random_tokens(rng, n_seq * WINDOW, shape.vocab).reshape(n_seq, WINDOW)
    cand[slot] = target
    if bad_token_of is not None:
        cand[bad_token_of, 0] = shape.vocab
    nv = None if n_valid is None else torch.as_tensor(n_valid.astype(np.int32), device=DEV)
    out, status, logits = sess.verify(kv, bt, torch.as_tensor(lens, device=DEV), torch.as_tensor(cand, device=DEV), n_valid=nv,
                                      dump_seq_ids=torch.tensor([slot], dtype=torch.int32, device=DEV),
                                      max_context=int(lens.max()) + WINDOW)
    torch.cuda.synchronize()
    assert status.tolist() == ([0] * n_seq if expect_status is None else expect_status)
    k, v = gpu_kv_tokens(kv, bt[slot], CONTEXT + WINDOW, shape.head_dim)
    return out.cpu(), logits[0].cpu(), k.cpu(), v.cpu()


@pytest.fixture(scope="module")
def alone(env):
    out, logits, k, v = _run(*env, 1, 0)
    assert torch.isfinite(logits).all()
    return out[0], logits, k, v


@pytest.mark.parametrize("n_seq", [2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 40, 41, 64, 65, 96, 97, 128, 160, 161, 192, 224, 256])
def test_same_bits_at_every_row_count(env, alone, n_seq):
    slot = n_seq - 1
    out, logits, k, v = _run(*env, n_seq, slot)
    assert torch.equal(out[slot], alone[0]) and int(out.min()) >= 0
    assert torch.equal(logits, alone[1]) and torch.equal(k, alone[2]) and torch.equal(v, alone[3])


@pytest.mark.parametrize("n_seq", [4, 5, 6, 7, 8, 9, 20, 41, 65, 97, 130, 200, 256, 300])
def test_same_bits_among_partly_filled_windows(env, alone, n_seq):
    """Partly filled windows are packed: the target's rows begin wherever the counts before it end (odd offsets, across
    tiles), sequences that fail a check have no rows or dead ones, and what lies behind the last row is skipped.  65 to 128 rows
    (5 - 8 sequences) take the 32 x 128 tile of partly filled windows for the split projections."""
    rng = wl.rng_for(47, 5, n_seq)
    n_valid = rng.integers(1, WINDOW + 1, size=n_seq)
    slot = n_seq - 2
    n_valid[slot] = WINDOW
    n_valid[0] = WINDOW + 1                                     # refused by its length: no rows
    expect = [0] * n_seq
    expect[0], expect[1] = B.LLM42_SEQ_BAD_LENGTH, B.LLM42_SEQ_BAD_TOKEN    # (the second one's rows are there, and dead)
    out, logits, k, v = _run(*env, n_seq, slot, n_valid, bad_token_of=1, expect_status=expect)
    assert torch.equal(out[slot], alone[0])
    assert torch.equal(logits, alone[1]) and torch.equal(k, alone[2]) and torch.equal(v, alone[3])
    live = torch.as_tensor(np.arange(WINDOW)[None, :] < n_valid[:, None])
    live[:2] = False
    assert bool(((out >= 0) == live).all())


_TOTALS = [32, 384, 512, 513, 576, 577, 640, 641, 704, 705, 768, 769, 1024]


@pytest.mark.parametrize("n_seq,total", [(48, t) for t in _TOTALS if t <= 768] + [(64, t) for t in _TOTALS] +
                         [(128, t) for t in (16, 1280, 1281, 2047, 2048)] + [(256, t) for t in (2304, 2305, 2560, 2561, 4096)])
def test_same_bits_on_both_sides_of_the_launch_for_fewer_rows(env, alone, n_seq, total):
    """Partly filled windows of 768 rows and more: a launch for no more rows than a multiple of 128 between 9/16 and 3/4 of
    all and one for more; exactly one of the two may run, whichever multiple it is.  (At 2048 rows the rule has it at 1280 for all
    four projections, at 4096 at 2304 for QKV and 2560 for O and down; the halves of those two follow each other there, so each
    side is two launches, the second of which adds the first one's partial.)"""
    slot = n_seq // 2
    n_valid = np.full(n_seq, 0)
    n_valid[slot] = WINDOW
    rest, others = total - WINDOW, [s for s in range(n_seq) if s != slot]
    for k, s in enumerate(others):
        n_valid[s] = (rest * (k + 1)) // len(others) - (rest * k) // len(others)
    expect = [0 if n else B.LLM42_SEQ_BAD_LENGTH for n in n_valid]           # (a count of 0 is refused: no rows)
    assert n_valid.sum() == total and n_valid.max() <= WINDOW
    out, logits, k, v = _run(*env, n_seq, slot, n_valid, expect_status=expect)
    assert torch.equal(out[slot], alone[0])
    assert torch.equal(logits, alone[1]) and torch.equal(k, alone[2]) and torch.equal(v, alone[3])


@pytest.mark.parametrize("d_model,n_kv_heads", [(1024, 2), (2048, 4)])
def test_same_bits_with_few_feature_blocks(d_model, n_kv_heads):
    """At most one block of 16 QKV features per CU: up to 64 rows a workgroup takes one block, not two; from 65 rows on the
    tiles of other kernels.  32 and 64 k-tiles, so every ring of the small-batch kernel is refilled."""
    shape = wl.LLAMA_8B.replace(n_layers=1, d_model=d_model, n_q_heads=16, n_kv_heads=n_kv_heads, head_dim=64, d_ffn=2048, vocab=1024)
    sess = VerifierSession(shape, wl.make_weights(shape, seed=49), max_position=128, device=DEV)
    want = _run(shape, sess, 5, 4)                              # 80 rows
    assert torch.isfinite(want[1]).all()
    for n_seq in (1, 2, 3, 4):
        out, logits, k, v = _run(shape, sess, n_seq, n_seq - 1)
        assert torch.equal(out[n_seq - 1], want[0][4]) and torch.equal(logits, want[1]), n_seq
        assert torch.equal(k, want[2]) and torch.equal(v, want[3]), n_seq
    sess.close()


@pytest.mark.parametrize("n_seq", [33, 48, 96])
@pytest.mark.parametrize("d_model", [1024, 2048, 8192])
def test_same_bits_with_norms_of_eight_rows_per_workgroup(d_model, n_seq):
    """Beyond 512 rows the norms of these widths are a kernel of their own that also adds the halves of the split projections
    (by the tile rule both projections leave theirs to it at 528 and 768 rows, and up to d_model 2048 at 1536)."""
    shape = wl.LLAMA_8B.replace(n_layers=1, d_model=d_model, n_q_heads=8, n_kv_heads=2, d_ffn=1024, vocab=1024)
    sess = VerifierSession(shape, wl.make_weights(shape, seed=53), max_position=128, device=DEV)
    want = _run(shape, sess, 1, 0)
    assert torch.isfinite(want[1]).all()
    n_valid = wl.rng_for(53, n_seq).integers(1, WINDOW + 1, size=n_seq)
    n_valid[n_seq - 1] = WINDOW
    for counts in (None, n_valid):
        out, logits, k, v = _run(shape, sess, n_seq, n_seq - 1, counts)
        assert torch.equal(out[n_seq - 1], want[0][0]) and torch.equal(logits, want[1])
        assert torch.equal(k, want[2]) and torch.equal(v, want[3])
    sess.close()


@pytest.fixture(scope="module")
def ragged():
    """28, 449 and 14 k-tiles (halves of 225 and 224, of 7 and 7), feature blocks that no tile divides: partial rounds and partial
    tiles in every kernel of more than 64 rows."""
    shape = wl.LLAMA_8B.replace(n_layers=1, d_model=896, n_q_heads=14, n_kv_heads=2, head_dim=64, d_ffn=14352, vocab=33296)
    sess = VerifierSession(shape, wl.make_weights(shape, seed=50), max_position=128, device=DEV)
    want = _run(shape, sess, 1, 0)                              # 16 rows: the small-batch kernels
    assert torch.isfinite(want[1]).all()
    yield shape, sess, want
    sess.close()


@pytest.mark.parametrize("n_seq", [5, 8, 12, 16, 24, 32, 40, 48, 56, 64, 72, 80, 96, 112, 128, 160, 192, 256])
def test_same_bits_with_partial_rounds_and_tiles(ragged, n_seq):
    shape, sess, want = ragged
    out, logits, k, v = _run(shape, sess, n_seq, n_seq - 1)
    assert torch.equal(out[n_seq - 1], want[0][0]) and torch.equal(logits, want[1])
    assert torch.equal(k, want[2]) and torch.equal(v, want[3])


@pytest.mark.parametrize("n_seq", [5, 8, 12, 16, 24, 32, 48, 64, 128])
def test_same_bits_with_partial_rounds_and_tiles_among_partly_filled_windows(ragged, n_seq):
    """Odd halves of the split projections by the 32 x 128 tile (5, 8, 16 - 32 sequences), and the LM head's tile of two
    workgroups per CU (from 32 sequences on) with rows left out."""
    shape, sess, want = ragged
    n_valid = wl.rng_for(50, n_seq).integers(1, WINDOW + 1, size=n_seq)
    n_valid[n_seq - 1] = WINDOW
    out, logits, k, v = _run(shape, sess, n_seq, n_seq - 1, n_valid)
    assert torch.equal(out[n_seq - 1], want[0][0]) and torch.equal(logits, want[1])
    assert torch.equal(k, want[2]) and torch.equal(v, want[3])


# Chosen by the tile rule: with the models above and the unsplit projections of test_gpu_batch_chosen.py, 122 of the 137 kernels of
# more than 64 rows (tile x epilogue, the sampled LM head aside) run in some test.
@pytest.mark.parametrize("d_model,heads,kv_heads,d_ffn,vocab,calls", [
    (256, 16, 8, 1024, 4096, [(24, False), (72, False)]),
    (256, 16, 2, 1024, 4096, [(80, False)]),
    (256, 16, 8, 2048, 4096, [(80, False)]),
    (256, 4, 2, 8192, 4096, [(5, False)]),
    (256, 32, 4, 1024, 4096, [(80, False)]),
    (768, 16, 8, 1024, 4096, [(48, False), (96, False)]),
    (1536, 32, 4, 1024, 4096, [(192, True)]),
    (1536, 4, 2, 1024, 4096, [(5, False)]),
    (1536, 4, 2, 1024, 33296, [(112, False)]),
    (1536, 4, 2, 1024, 50304, [(40, False)]),
    (3072, 4, 2, 1024, 4096, [(24, False), (32, False), (112, False), (128, False), (320, False)]),
    (3072, 4, 2, 1024, 16384, [(72, False)]),
    (3072, 32, 4, 1024, 4096, [(256, True)]),
])
def test_same_bits_by_the_other_tiles(d_model, heads, kv_heads, d_ffn, vocab, calls):
    shape = wl.LLAMA_8B.replace(n_layers=1, d_model=d_model, n_q_heads=heads, n_kv_heads=kv_heads, d_ffn=d_ffn, vocab=vocab)
    sess = VerifierSession(shape, wl.make_weights(shape, seed=54), max_position=128, device=DEV)
    want = _run(shape, sess, 1, 0)
    assert torch.isfinite(want[1]).all()
    for n_seq, partly in calls:
        n_valid = wl.rng_for(54, n_seq).integers(1, WINDOW + 1, size=n_seq)
        n_valid[n_seq - 1] = WINDOW
        out, logits, k, v = _run(shape, sess, n_seq, n_seq - 1, n_valid if partly else None)
        assert torch.equal(out[n_seq - 1], want[0][0]) and torch.equal(logits, want[1])
        assert torch.equal(k, want[2]) and torch.equal(v, want[3])
    sess.close()


@pytest.mark.timeout(300)
def test_partly_filled_windows_as_whole_sequence_items():
    shape = wl.TINY
    sess = VerifierSession(shape, wl.make_weights(shape, seed=48), max_position=2400, device=DEV)
    window, slot, L = 64, 131, 2200
    target = wl.random_tokens(wl.rng_for(48, 1), window, shape.vocab)

    def run(n_seq, slot):
        rng = wl.rng_for(48, 2, n_seq)
        lens = rng.integers(2150, 2250, size=n_seq).astype(np.int32)
        lens[slot] = L
        n_valid = rng.integers(1, window + 1, size=n_seq).astype(np.int32)
        n_valid[slot] = 41
        table, blocks = wl.make_block_table(rng, lens + window, 16, spare_blocks=2)
        bt = torch.as_tensor(table, device=DEV)
        kv = sess.kv_cache(blocks)
        kv.normal_(generator=torch.Generator(device=DEV).manual_seed(n_seq))
        mine = torch.empty((shape.n_layers, 2, 142, shape.n_kv_heads, 16 * shape.head_dim), dtype=torch.bfloat16, device=DEV)
        kv[:, :, bt[slot, :142].long()] = mine.normal_(generator=torch.Generator(device=DEV).manual_seed(7))
        cand = wl.random_tokens(rng, n_seq * window, shape.vocab).reshape(n_seq, window)
        cand[slot] = target
        d = lambda a: torch.as_tensor(a, device=DEV)
        mc = int(lens.max()) + window
        out, status, logits = sess.verify(kv, bt, d(lens), d(cand), n_valid=d(n_valid), max_context=mc,
                                          dump_seq_ids=torch.tensor([slot], dtype=torch.int32, device=DEV))
        torch.cuda.synchronize()
        assert int(status.max()) == 0
        plan = B.llm42_measure_attention_plan(sess.model, n_seq, window, mc)
        if plan["may_take_sequences"]:
            flag = sess.workspace(n_seq, window, mc)[plan["sequences_flag_offset"]:plan["sequences_flag_offset"] + 4]
            assert int(flag.view(torch.int32)[0]) == 1
        return out[slot].cpu(), logits[0, :41].cpu(), plan["may_take_sequences"]

    few, many = run(1, 0), run(256, slot)
    assert many[2] and not few[2]
    assert torch.equal(few[0], many[0]) and torch.equal(few[1], many[1])
    sess.close()


def test_partly_filled_windows_of_more_sequences_than_are_packed():
    """Beyond 4096 sequences the rows are not packed: padding rows stay where they are, with zeros for their attention output."""
    shape = wl.TINY
    sess = VerifierSession(shape, wl.make_weights(shape, seed=50), max_position=64, device=DEV)
    n_seq, window = 4100, 4
    rng = wl.rng_for(50, 1)
    lens = rng.integers(0, 40, size=n_seq).astype(np.int32)
    n_valid = rng.integers(1, window + 1, size=n_seq).astype(np.int32)
    n_valid[3], sample = 0, [0, 1, 2, 2000, 4095, 4096, 4099]     # (a count of 0 is refused)
    table, blocks = wl.make_block_table(rng, lens + window, 16, spare_blocks=2)
    bt = torch.as_tensor(table, device=DEV)
    kv = sess.kv_cache(blocks)
    kv.normal_(generator=torch.Generator(device=DEV).manual_seed(5))
    cand = wl.random_tokens(rng, n_seq * window, shape.vocab).reshape(n_seq, window)
    d = lambda a: torch.as_tensor(a, device=DEV)
    out, status, logits = sess.verify(kv, bt, d(lens), d(cand), n_valid=d(n_valid),
                                      dump_seq_ids=torch.tensor(sample, dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    assert status.nonzero().flatten().tolist() == [3] and int(status[3]) == B.LLM42_SEQ_BAD_LENGTH
    taken = torch.as_tensor(np.arange(window)[None, :] < n_valid[:, None])
    assert bool(((out.cpu() >= 0) == taken).all())
    for j, s in enumerate(sample):
        n = int(n_valid[s])
        one, _, alone = sess.verify(kv, bt[s:s + 1].contiguous(), d(lens[s:s + 1]), d(cand[s:s + 1]), n_valid=d(n_valid[s:s + 1]),
                                    dump_seq_ids=torch.zeros(1, dtype=torch.int32, device=DEV))
        torch.cuda.synchronize()
        assert torch.equal(alone[0, :n], logits[j, :n]) and torch.equal(one[0], out[s]), s
    sess.close()


@pytest.mark.parametrize("n_seq", [9, 41, 97])
def test_same_bits_when_the_last_sequence_is_refused(env, alone, n_seq):
    """Where the packed rows end is read from the last sequence's tag: refused for its length (no rows), then for a token."""
    rng = wl.rng_for(47, 6, n_seq)
    n_valid = rng.integers(1, WINDOW + 1, size=n_seq)
    slot = n_seq - 2
    n_valid[slot] = WINDOW
    for code in (B.LLM42_SEQ_BAD_LENGTH, B.LLM42_SEQ_BAD_TOKEN):
        n_valid[-1] = 0 if code == B.LLM42_SEQ_BAD_LENGTH else 7
        expect = [0] * (n_seq - 1) + [code]
        out, logits, k, v = _run(*env, n_seq, slot, n_valid, bad_token_of=n_seq - 1 if code == B.LLM42_SEQ_BAD_TOKEN else None,
                                 expect_status=expect)
        assert torch.equal(out[slot], alone[0]) and int(out[-1].max()) == -1
        assert torch.equal(logits, alone[1]) and torch.equal(k, alone[2]) and torch.equal(v, alone[3])
