"""Windows of several groups of 128 query rows where the query heads per kv head do not divide 128, partly filled: the rows of a group
then span a number of tokens that is no whole one, and each group has the keys of its own last token.  The same rows in windows of at
most 16 tokens, one sequence at a time, give the same bits."""
import numpy as np
import pytest
import torch

from helpers import wl
from gpu_helpers import VerifierSession
from paper_2601_17768_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("group,window", [(3, 80), (3, 129), (5, 52), (6, 64), (7, 40), (7, 111)])
def test_same_bits_as_in_small_windows(group, window, head_dim):
    shape = wl.TINY.replace(n_q_heads=2 * group, n_kv_heads=2, head_dim=head_dim)
    sess = VerifierSession(shape, wl.make_weights(shape, seed=61), max_position=2600, device=DEV)
    rng = wl.rng_for(61, group, window, head_dim)
    # beyond one super and within; last tokens around the edges of a step behind 128 / group, 256 / group, ... tokens
    lens = np.array([2040 - 128 // group, 2100, 0, 64 - 128 // group, 700, 255, 63], dtype=np.int32)
    rows = np.array([window, window - 1, window, window, 128 // group + 1, min(window, 128 // group), 1], dtype=np.int32)
    n = len(lens)
    table, blocks = wl.make_block_table(rng, lens + window, 16, spare_blocks=2)
    d = lambda a: torch.as_tensor(a, device=DEV)
    bt, sl, nv = d(table), d(lens), d(rows)
    cand = wl.random_tokens(rng, n * window, shape.vocab).reshape(n, window)
    kv0 = sess.kv_cache(blocks)
    kv0.normal_(generator=torch.Generator(device=DEV).manual_seed(6))
    for s in range(n):                                                     # nothing behind a context is ever read
        last = (int(lens[s]) + window + 15) // 16
        kv0[:, :, bt[s, (int(lens[s]) + 15) // 16:last].long()] = float("nan")
    kv, each = kv0.clone(), kv0.clone()
    max_context = int(lens.max()) + window
    assert B.llm42_measure_attention_plan(sess.model, n, window, max_context)["streaming"]
    out, status, logits = sess.verify(kv, bt, sl, d(cand), n_valid=nv, max_context=max_context,
                                      dump_seq_ids=torch.arange(n, dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    assert int(status.abs().max()) == 0
    for s in range(n):
        for i in range(0, int(rows[s]), 16):
            k = min(16, int(rows[s]) - i)
            o, st, lg = sess.verify(each, bt[s:s + 1].contiguous(), d(np.array([lens[s] + i], dtype=np.int32)),
                                    d(np.ascontiguousarray(cand[s:s + 1, i:i + k])), max_context=int(lens[s]) + i + k,
                                    dump_seq_ids=torch.zeros(1, dtype=torch.int32, device=DEV))
            torch.cuda.synchronize()
            assert int(st[0]) == 0 and torch.isfinite(lg).all()
            assert torch.equal(out[s, i:i + k], o[0]) and torch.equal(logits[s, i:i + k], lg[0])
    assert torch.equal(kv.view(torch.int16), each.view(torch.int16))
    sess.close()
