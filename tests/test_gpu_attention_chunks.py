"""Attention by chunks of 256 keys at head dimension 128: which calls of 8 and more blocks of query rows run it with 4 waves and two
workgroups to a CU instead of 8 waves and one, and calls in which such a workgroup walks several items."""
import numpy as np
import pytest
import torch

from helpers import wl
from gpu_helpers import VerifierSession
from paper_2601_17768_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SHAPE = wl.TINY.replace(d_model=512, n_q_heads=32, n_kv_heads=8, head_dim=128)


@pytest.fixture(scope="module")
def sess():
    s = VerifierSession(SHAPE, wl.make_weights(SHAPE, seed=59), max_position=9000, device=DEV)
    yield s
    s.close()


# sequences, window, longest context: measured to be slower by 4 waves, or not
SLOWER = [(1, 32, 4532), (1, 32, 8032), (2, 32, 1932), (2, 32, 3032), (4, 32, 1932), (1, 64, 3064), (2, 64, 1964), (1, 128, 1928)]
FASTER = [(1, 32, 1932), (1, 64, 1564), (3, 32, 1032), (4, 32, 544), (4, 32, 1032), (5, 32, 332), (8, 32, 332), (1, 256, 768), (1, 48, 4548)]


@pytest.mark.parametrize("n,window,max_context,streaming", [(*c, True) for c in SLOWER] + [(*c, False) for c in FASTER])
def test_four_waves_only_where_they_are_not_slower(sess, n, window, max_context, streaming):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("measured with 256 CUs")
    plan = B.llm42_measure_attention_plan(sess.model, n, window, max_context)
    assert plan["item_keys"] == 256 and not plan["split"] and plan["streaming"] == streaming


@pytest.mark.parametrize("window,ragged,alone", [(8, False, 11), (8, True, 11), (16, True, 11), (28, False, 5)])
def test_several_chunks_per_workgroup(sess, window, ragged, alone):
    """2, 4 and 7 blocks of query rows (two groups of four), 11 or 5 sequences of up to 4096 keys: more than two items for each of two
    workgroups to a CU, of one step to four.  Among more sequences the call runs per super; the schedule is fixed, so the bits are the same."""
    rng = wl.rng_for(59, window, int(ragged))
    top = 4096 - window
    lens = np.concatenate([[top, top - 1, 3839, 3840, 3841, 3900, 3903, 3904, 3968, 4030, 4000], rng.integers(0, 300, size=16)]).astype(np.int32)
    rows = rng.integers(1, window + 1, size=len(lens)).astype(np.int32) if ragged else np.full(len(lens), window, dtype=np.int32)
    table, blocks = wl.make_block_table(rng, lens + window, 16, spare_blocks=2)
    d = lambda a: torch.as_tensor(a, device=DEV)
    bt, sl, nv = d(table), d(lens), d(rows)
    cand = d(wl.random_tokens(rng, len(lens) * window, SHAPE.vocab).reshape(-1, window))
    kv0 = sess.kv_cache(blocks)
    kv0.normal_(generator=torch.Generator(device=DEV).manual_seed(5))
    max_context = 4096

    def run(n):
        plan = B.llm42_measure_attention_plan(sess.model, n, window, max_context)
        ws = torch.empty(B.llm42_workspace_bytes(sess.model, n, window, max_context), dtype=torch.uint8, device=DEV)
        kv, out = kv0.clone(), torch.full((n, window), -1, dtype=torch.int32, device=DEV)
        logits = torch.zeros((alone, window, SHAPE.vocab), device=DEV)
        B.llm42_verify_window(sess.model, kv, blocks, bt[:n].contiguous(), sl[:n].contiguous(), cand[:n].contiguous(), window,
                              nv[:n].contiguous() if ragged else None, max_context, out, ws, None, logits,
                              torch.arange(alone, dtype=torch.int32, device=DEV))
        torch.cuda.synchronize()
        at = plan["sequences_flag_offset"] - 4 * (1 + SHAPE.n_layers)      # the number of listed items (see test_gpu_attention_waves.py)
        return plan, int(ws[at:at + 4].view(torch.int32)[0]), out[:alone].clone(), logits

    few, many = run(alone), run(len(lens))
    assert few[0]["item_keys"] == 256 and not few[0]["streaming"] and not few[0]["split"] and not few[0]["waves"]
    assert few[1] * SHAPE.n_kv_heads * ((window * 4 + 63) // 64) > 2 * 2 * torch.cuda.get_device_properties(0).multi_processor_count
    assert many[0]["item_keys"] == 2048 and torch.isfinite(few[3]).all()
    assert torch.equal(few[2], many[2]) and torch.equal(few[3], many[3])
