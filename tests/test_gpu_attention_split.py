"""The attention kernel for few row blocks (a workgroup per 16 query rows, chunks of 256 keys dealt to its waves) gives
the same bits as the kernels that take over when more sequences share the call, at contexts around the edges of its
steps, chunks and waves.  Those kernels are held to the checker in test_gpu_attention_modes.py; the schedule is fixed,
so the comparison is exact."""
import numpy as np
import pytest
import torch

from helpers import wl
from gpu_helpers import VerifierSession
from paper_2601_17768_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SHAPES = {64: wl.TINY, 128: wl.TINY.replace(d_model=512, n_q_heads=4, n_kv_heads=1, head_dim=128)}


@pytest.fixture(scope="module", params=[64, 128])
def env(request):
    shape = SHAPES[request.param]
    sess = VerifierSession(shape, wl.make_weights(shape, seed=51), max_position=2048, device=DEV)
    yield shape, sess
    sess.close()


def _run(shape, sess, L, window, rows, others, other_len, max_context, split=None):
    """Target first among `others` sequences of `other_len` cached keys; its cache is the same in every company and
    holds NaN behind its last position."""
    rng = wl.rng_for(51, L, window)
    cand_t = wl.random_tokens(rng, window, shape.vocab)
    lens = np.array([L] + [other_len] * others, dtype=np.int32)
    table, blocks = wl.make_block_table(wl.rng_for(51, others), lens + window, 16, spare_blocks=2)
    wide = np.full((1 + others, 128), -7, dtype=np.int32)      # entries past a sequence's blocks may hold anything
    wide[:, :table.shape[1]] = table
    bt = torch.as_tensor(wide, device=DEV)
    kv = sess.kv_cache(blocks)
    kv.normal_(generator=torch.Generator(device=DEV).manual_seed(1))
    nb = (L + window + 15) // 16
    mine = torch.empty((shape.n_layers, 2, nb, shape.n_kv_heads, 16 * shape.head_dim), dtype=torch.bfloat16, device=DEV)
    mine.normal_(generator=torch.Generator(device=DEV).manual_seed(2))
    mine[:, :, (L + 15) // 16:] = float("nan")
    kv[:, :, bt[0, :nb].long()] = mine
    cand = wl.random_tokens(wl.rng_for(51, 9), (1 + others) * window, shape.vocab).reshape(1 + others, window)
    cand[0] = cand_t
    nv = np.full(1 + others, window, dtype=np.int32)
    nv[0] = rows
    if split is not None:
        assert B.llm42_measure_attention_plan(sess.model, 1 + others, window, max_context)["split"] == split
    d = lambda a: torch.as_tensor(a, device=DEV)
    out, status, logits = sess.verify(kv, bt, d(lens), d(cand), n_valid=d(nv), max_context=max_context,
                                      dump_seq_ids=torch.zeros(1, dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    assert int(status.max()) == 0
    return out[0].cpu(), logits[0, :rows].cpu()


@pytest.mark.parametrize("L", [0, 1, 15, 47, 63, 64, 240, 255, 256, 500, 1000, 1023, 1024, 1270])
@pytest.mark.parametrize("window,rows", [(1, 1), (8, 8), (9, 5), (33, 33)])
def test_same_bits_as_in_a_large_group(env, L, window, rows):
    if L + window > 1280 and window > 8:
        pytest.skip("such a call takes the other kernels anyway")
    shape, sess = env
    # alone, bounded tightly: the split kernel; behind a bound beyond one super: chunk items and the merge pass
    alone = _run(shape, sess, L, window, rows, 0, 0, max(L + window, 16), split=True)
    merged = _run(shape, sess, L, window, rows, 0, 0, 2048 if L + window > 1280 else 1281, split=False)
    assert torch.isfinite(alone[1]).all()
    assert torch.equal(alone[0], merged[0]) and torch.equal(alone[1], merged[1])
    # several items per workgroup of the split kernel (300 sequences x 1-2 kv heads > 256), or the other kernels
    crowd = _run(shape, sess, L, window, rows, 300, 20, max(L, 20) + window)
    assert torch.equal(alone[0], crowd[0]) and torch.equal(alone[1], crowd[1])


def one_block(shape, window):
    """Fewer sequences of one row block at head dimension 128 take a wave per chunk at such contexts (test_gpu_attention_waves.py)."""
    return shape.head_dim == 128 and window == 1


@pytest.mark.parametrize("L", [1279, 1281, 1535, 1536, 1791, 1792, 2040])
@pytest.mark.parametrize("window,rows", [(1, 1), (8, 8), (8, 3)])
def test_second_chunk_of_every_wave(env, L, window, rows):
    """Contexts of six to eight chunks: each wave walks two.  Enough company that the call takes the split kernel at such
    contexts; alone they go through chunk items and the merge pass."""
    shape, sess = env
    merged = _run(shape, sess, L, window, rows, 0, 0, max(L + window, 1281), split=False)
    assert torch.isfinite(merged[1]).all()
    among = _run(shape, sess, L, window, rows, 239 if one_block(shape, window) else 60, 20, L + window, split=True)
    assert torch.equal(merged[0], among[0]) and torch.equal(merged[1], among[1])


@pytest.mark.parametrize("L", [1281, 1536, 1791, 2040])
def test_second_chunk_of_items_from_the_list(env, L):
    """One row block and more workgroups than CUs: the split kernel takes its items from the plan's list."""
    shape, sess = env
    if shape.head_dim != 128:
        pytest.skip("the other kernels take such a call at head dimension 64")
    merged = _run(shape, sess, L, 4, 3, 0, 0, L + 4, split=False)
    listed = _run(shape, sess, L, 4, 3, 400, 20, L + 4, split=True)
    assert torch.equal(merged[0], listed[0]) and torch.equal(merged[1], listed[1])
