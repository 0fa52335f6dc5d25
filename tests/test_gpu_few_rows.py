"""Passes of up to 64 rows fetch only the activation rows that there are: at row counts around the edges of a line (8 rows), a
token block (16) and a pass's padding (16, 32, 64) every row has the bits that it has among more sequences.  The larger group
takes other GEMM kernels; those are held to the oracle elsewhere, and the schedule is fixed, so the comparison is exact."""
import numpy as np
import pytest
import torch

from helpers import wl
from gpu_helpers import VerifierSession

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SHAPE = wl.TINY.replace(d_model=640, n_q_heads=8, n_kv_heads=2, d_ffn=1008)     # k-tiles: 20, 16 and 32, rounds with and without a rest
MOST = 80


@pytest.fixture(scope="module")
def env():
    sess = VerifierSession(SHAPE, wl.make_weights(SHAPE, seed=54), max_position=128, device=DEV)
    rng = wl.rng_for(54, 1)
    lens = rng.integers(0, 60, size=MOST).astype(np.int32)
    table, blocks = wl.make_block_table(rng, lens + 1, 16, spare_blocks=1)
    bt, sl = torch.as_tensor(table, device=DEV), torch.as_tensor(lens, device=DEV)
    kv = sess.kv_cache(blocks)
    kv.normal_(generator=torch.Generator(device=DEV).manual_seed(4))
    cand = torch.as_tensor(wl.random_tokens(rng, MOST, SHAPE.vocab).reshape(MOST, 1), device=DEV)

    def run(n):
        mine = kv.clone()
        out, status, logits = sess.verify(mine, bt[:n].contiguous(), sl[:n].contiguous(), cand[:n].contiguous(),
                                          dump_seq_ids=torch.arange(n, dtype=torch.int32, device=DEV))
        torch.cuda.synchronize()
        assert int(status.max()) == 0
        return out.cpu(), logits.cpu()

    yield run, run(MOST)
    sess.close()


@pytest.mark.parametrize("rows", [1, 2, 7, 8, 9, 15, 16, 17, 24, 25, 31, 32, 33, 40, 47, 48, 49, 63, 64])
def test_same_bits_as_among_more_rows(env, rows):
    run, (tokens, logits) = env
    t, l = run(rows)
    assert torch.isfinite(l).all()
    assert torch.equal(t, tokens[:rows]) and torch.equal(l, logits[:rows])
