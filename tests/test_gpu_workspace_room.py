"""What a call's workspace must hold: the least that is accepted, and what llm42_workspace_bytes counts."""
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
    s = VerifierSession(SHAPE, wl.make_weights(SHAPE, seed=58), max_position=9000, device=DEV)
    yield s
    s.close()


def _call(sess, lens, window, max_context):
    """The verify call of these cached lengths as a function of its workspace; returns its tokens."""
    n = len(lens)
    lens = np.asarray(lens, dtype=np.int32)
    rng = wl.rng_for(58, n, window)
    table, blocks = wl.make_block_table(rng, lens + window, 16, max_blocks_per_seq=(max_context + 15) // 16, spare_blocks=1)
    d = lambda a: torch.as_tensor(a, device=DEV)
    bt, sl = d(table), d(lens)
    cand = d(wl.random_tokens(rng, n * window, SHAPE.vocab).reshape(n, window))
    kv = sess.kv_cache(blocks)
    kv.normal_(generator=torch.Generator(device=DEV).manual_seed(3))
    out = torch.full((n, window), -7, dtype=torch.int32, device=DEV)

    def run(ws):
        B.llm42_verify_window(sess.model, kv, blocks, bt, sl, cand, window, None, max_context, out, ws)
        torch.cuda.synchronize()
        return out.clone()

    return run


@pytest.mark.parametrize("lens,window,max_context", [([2048, 4100], 1, 4101), ([300] * 11, 1, 2001), ([9, 20, 4100], 2, 4102)])
def test_the_least_workspace_is_that_of_the_work_split_without_a_wave_per_chunk(sess, lens, window, max_context):
    """Calls that run per 256-key chunk for every number of sequences up to theirs: llm42_workspace_bytes is exactly what they
    need.  A wave per chunk would do with less (its slots have as many rows as there are query rows, not padded to 16)."""
    need = B.llm42_workspace_bytes(sess.model, len(lens), window, max_context)
    run = _call(sess, lens, window, max_context)
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    with pytest.raises(B.Llm42Error) as e:
        run(ws[:need - 256])
    assert e.value.status == B.LLM42_EWORKSPACE
    assert int(run(ws).min()) >= 0


@pytest.mark.parametrize("n,window,max_context", [(40, 4, 2044), (40, 3, 1500)])
def test_workspace_bytes_has_room_for_a_wave_per_chunk(sess, n, window, max_context):
    """One block of query rows and more sequences than a workgroup each would fit the device: the calls that run a wave per
    256-key chunk, with a partial of every query row (accumulators, maximum and sum in 32 bits) per chunk."""
    rows, chunks = 4 * window, (max_context + 255) // 256
    partials = n * SHAPE.n_kv_heads * chunks * rows * (SHAPE.head_dim * 4 + 8)
    queries = n * SHAPE.n_kv_heads * 16 * SHAPE.head_dim * 2
    assert B.llm42_workspace_bytes(sess.model, n, window, max_context) >= partials + queries
    for fewer in (1, n // 2, n - 1):
        assert B.llm42_workspace_bytes(sess.model, fewer, window, max_context) <= B.llm42_workspace_bytes(sess.model, n, window, max_context)
