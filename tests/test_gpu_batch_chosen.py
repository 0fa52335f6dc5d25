"""The residual projections without their k-split (the fast path beyond 16 rows, llm42_measure_verify_window_batch_chosen), by
value at widths that go several times round the rings of their kernels.  Unsplit, an element is one accumulator over
ascending k whatever kernel computes it, so 32-, 64- and 128-row passes give the same bits; and the fixed schedule's logits
differ by rounding only."""
import numpy as np
import pytest
import torch

from helpers import wl
from gpu_helpers import VerifierSession
from paper_2601_17768_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CONTEXT = 40


def _logits(shape, sess, n_seq, window, batch_chosen):
    """Logits of the last sequence of the call, whose tokens and cache are the same in every call of this window."""
    rng = wl.rng_for(61, window)
    target = wl.random_tokens(rng, window, shape.vocab)
    nb = (CONTEXT + window + 15) // 16
    mine = torch.empty((1, 2, nb, shape.n_kv_heads, 16 * shape.head_dim), dtype=torch.bfloat16, device=DEV)
    mine.normal_(generator=torch.Generator(device=DEV).manual_seed(1))
    rng = wl.rng_for(61, window, n_seq)
    lens = rng.integers(1, 60, size=n_seq).astype(np.int32)
    lens[-1] = CONTEXT
    table, blocks = wl.make_block_table(rng, lens + window, 16, spare_blocks=2)
    bt = torch.as_tensor(table, device=DEV)
    kv = sess.kv_cache(blocks)
    kv.normal_(generator=torch.Generator(device=DEV).manual_seed(n_seq))
    kv[:, :, bt[-1, :nb].long()] = mine
    cand = wl.random_tokens(rng, n_seq * window, shape.vocab).reshape(n_seq, window)
    cand[-1] = target
    d = lambda a: torch.as_tensor(a, device=DEV)
    out = torch.empty((n_seq, window), dtype=torch.int32, device=DEV)
    logits = torch.empty((1, window, shape.vocab), dtype=torch.float32, device=DEV)
    max_context = int(lens.max()) + window
    B.llm42_verify_window(sess.model, kv, blocks, bt, d(lens), d(cand), window, None, max_context, out,
                          sess.workspace(n_seq, window, max_context), None, logits, torch.tensor([n_seq - 1], dtype=torch.int32, device=DEV),
                          batch_chosen=batch_chosen)
    torch.cuda.synchronize()
    assert torch.equal(out[-1].long(), logits[0].argmax(dim=1))
    return logits[0].cpu()


# 4096: a workgroup per block of 16 output features (128 k-tiles of the O-projection are 8 rounds of the ring, 448 of the
# down-projection 28); 4224: more blocks than CUs, two per workgroup
@pytest.mark.timeout(300)
@pytest.mark.parametrize("d_model,d_ffn", [(4096, 14336), (4224, 2064)])
def test_unsplit_projections_by_value(d_model, d_ffn):
    shape = wl.LLAMA_8B.replace(n_layers=1, d_model=d_model, d_ffn=d_ffn, vocab=2048)
    sess = VerifierSession(shape, wl.make_weights(shape, seed=61), max_position=128, device=DEV)
    for window, counts in ((17, (1, 3)), (16, (2, 3, 4)), (1, (17, 32, 33, 64))):
        want = _logits(shape, sess, 128 // window, window, True)            # 119 or 128 rows: the tiled kernels
        fixed = _logits(shape, sess, 128 // window, window, False)
        gap = (want - fixed).double()
        rel, worst = float(gap.norm() / fixed.double().norm()), float(gap.abs().max() / fixed.double().pow(2).mean().sqrt())
        print(f"d_model {d_model} window {window}: unsplit against split, 2-norm {rel:.2e}, largest over rms {worst:.2e}")
        for n_seq in counts:
            assert torch.equal(_logits(shape, sess, n_seq, window, True), want), (window, n_seq)
        # A last bit of a sum turns into a rounding (2^-9) of some of the bf16 values that follow; measured up to 8.1e-4 and
        # 8.4e-3, bounded at about four times that.  A stale or missing k-tile moves the logits by the order of their size.
        assert rel <= 3e-3 and worst <= 3e-2
    sess.close()


@pytest.mark.parametrize("d_model", [768, 2048])
def test_unsplit_projections_of_many_rows(d_model):
    """One accumulator per element whatever the tile: the same bits from 32 to 4096 rows."""
    shape = wl.LLAMA_8B.replace(n_layers=1, d_model=d_model, n_q_heads=16, n_kv_heads=8, d_ffn=2064, vocab=2048)
    sess = VerifierSession(shape, wl.make_weights(shape, seed=62), max_position=128, device=DEV)
    want = _logits(shape, sess, 2, 16, True)
    assert torch.isfinite(want).all()
    for n_seq in (5, 12, 16, 24, 32, 40, 48, 56, 64, 72, 80, 96, 128, 192, 256):
        assert torch.equal(_logits(shape, sess, n_seq, 16, True), want), n_seq
    sess.close()
