"""Calls without counts, whose windows are all full, run attention by 8 waves without the tests for rows that are not there; the
same windows given as counts run it with them.  The schedule is fixed, so both give the same bits, in every distribution of the work."""
import numpy as np
import pytest
import torch

from helpers import wl
from gpu_helpers import VerifierSession
from paper_2601_17768_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SHAPES = {64: wl.TINY.replace(n_q_heads=8, n_kv_heads=2), 128: wl.TINY.replace(d_model=512, n_q_heads=32, n_kv_heads=8, head_dim=128)}


@pytest.fixture(scope="module", params=[64, 128])
def env(request):
    shape = SHAPES[request.param]
    sess = VerifierSession(shape, wl.make_weights(shape, seed=60), max_position=4608, device=DEV)
    yield shape, sess
    sess.close()


# window, cached lengths (or how many from .. to); 4 query heads per kv head: 1, 2, 2 and 4 groups of 128 rows
CASES = [(32, [0, 1, 31, 32, 33, 63, 64, 1000, 2015, 2016] * 2), (32, [2015, 2016, 2017, 4100, 100]), (32, "uniform:100:2000:70"),
         (32, "uniform:2040:2300:40"), (64, [4100]), (64, "uniform:4000:4100:256"), (64, "uniform:0:1980:30"), (64, [1984, 1985, 2049]),
         (128, [1000, 1500, 2200]), (128, "uniform:900:1900:16")]


@pytest.mark.parametrize("window,lens", CASES, ids=[str(c)[:40] for c in CASES])
def test_same_bits_as_with_counts(env, window, lens):
    shape, sess = env
    rng = wl.rng_for(60, window, len(lens))
    if isinstance(lens, str):
        _, lo, hi, n = lens.split(":")
        lens = rng.integers(int(lo), int(hi) + 1, size=int(n))
    lens = np.array(lens, dtype=np.int32)
    n = len(lens)
    table, blocks = wl.make_block_table(rng, lens + window, 16, spare_blocks=2)
    d = lambda a: torch.as_tensor(a, device=DEV)
    bt, sl = d(table), d(lens)
    cand = d(wl.random_tokens(rng, n * window, shape.vocab).reshape(n, window))
    kv0 = sess.kv_cache(blocks)
    kv0.normal_(generator=torch.Generator(device=DEV).manual_seed(4))
    dump = torch.arange(0, n, max(1, n // 8), dtype=torch.int32, device=DEV)
    got = []
    for counts in (None, d(np.full(n, window, dtype=np.int32))):
        kv = kv0.clone()
        out, status, logits = sess.verify(kv, bt, sl, cand, n_valid=counts, max_context=int(lens.max()) + window, dump_seq_ids=dump)
        torch.cuda.synchronize()
        assert int(status.abs().max()) == 0 and torch.isfinite(logits).all()
        got.append((out.clone(), logits.clone(), kv))
    assert B.llm42_measure_attention_plan(sess.model, n, window, int(lens.max()) + window)["streaming"]
    for a, b in zip(*got):
        assert torch.equal(a, b)
