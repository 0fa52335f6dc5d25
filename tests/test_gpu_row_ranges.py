"""Logits and new K / V of a sequence are the same bits at every row count of a pass, at the 8B model's layer
widths (one layer): the row counts below lie on both sides of every line at which a kernel changes its tile or its
rows per workgroup.  The reference is the sequence verified alone, which test_gpu_mid.py holds to the oracle; the
reduction schedule is part of the interface, so the comparison is exact."""
import numpy as np
import pytest
import torch

from helpers import wl
from gpu_helpers import VerifierSession, gpu_kv_tokens

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
WINDOW, CONTEXT = 16, 40


@pytest.fixture(scope="module")
def env():
    shape = wl.LLAMA_8B.replace(n_layers=1, vocab=4096)
    sess = VerifierSession(shape, wl.make_weights(shape, seed=47), max_position=128, device=DEV)
    yield shape, sess
    sess.close()


def _run(shape, sess, n_seq, slot, n_valid=None):
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
    nv = None if n_valid is None else torch.as_tensor(n_valid.astype(np.int32), device=DEV)
    out, status, logits = sess.verify(kv, bt, torch.as_tensor(lens, device=DEV), torch.as_tensor(cand, device=DEV), n_valid=nv,
                                      dump_seq_ids=torch.tensor([slot], dtype=torch.int32, device=DEV),
                                      max_context=int(lens.max()) + WINDOW)
    torch.cuda.synchronize()
    assert int(status.max()) == 0
    k, v = gpu_kv_tokens(kv, bt[slot], CONTEXT + WINDOW, shape.head_dim)
    return out.cpu(), logits[0].cpu(), k.cpu(), v.cpu()


@pytest.fixture(scope="module")
def alone(env):
    out, logits, k, v = _run(*env, 1, 0)
    assert torch.isfinite(logits).all()
    return out[0], logits, k, v


@pytest.mark.parametrize("n_seq", [2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 40, 41, 64, 65, 96, 97, 128, 160, 161])
def test_same_bits_at_every_row_count(env, alone, n_seq):
    slot = n_seq - 1
    out, logits, k, v = _run(*env, n_seq, slot)
    assert torch.equal(out[slot], alone[0]) and int(out.min()) >= 0
    assert torch.equal(logits, alone[1]) and torch.equal(k, alone[2]) and torch.equal(v, alone[3])
