"""The attention kernel of decode steps and of windows of a few rows (a wave per 256-key chunk, one block of 16 query rows per
sequence and kv head) gives the same bits as the kernels that such a call runs when its workspace has no room for a partial of
every chunk.  Those are held to the checker in test_gpu_attention_modes.py; the schedule is fixed, so the comparison is exact."""
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
    s = VerifierSession(SHAPE, wl.make_weights(SHAPE, seed=53), max_position=4608, device=DEV)
    yield s
    s.close()


def _least(call, bytes_):
    """The smallest workspace that the call accepts (it is refused on the host, before anything runs)."""
    lo, hi = 0, bytes_ // 256
    while lo + 1 < hi:
        mid = (lo + hi) // 2
        try:
            call(mid * 256)
            hi = mid
        except B.Llm42Error:
            lo = mid
    return hi * 256


# chunk and step edges: contexts of one chunk (no merge), of whole chunks, of a last chunk of one to four steps, past one super;
# sequences x 8 kv heads: fewer items than waves, several per wave with short ones last (1024 waves), windows of one and four rows
CASES = [(1, [2047]), (1, [2048, 4100]), (1, [0, 254, 255, 256, 257, 319, 320, 511, 512, 1023, 2000]), (4, [0, 251, 252, 253, 508, 2044, 2045, 4200]),
         (1, "uniform:0:1300:17"), (1, "uniform:0:700:60"), (4, "uniform:1:2100:40"), (1, "uniform:4000:4500:12"), (1, "uniform:257:300:150")]


@pytest.mark.parametrize("window,lens", CASES, ids=[str(c) for c in CASES])
def test_same_bits_with_and_without_room_for_the_partials(sess, window, lens):
    rng = wl.rng_for(53, window, len(lens))
    if isinstance(lens, str):
        _, lo, hi, n = lens.split(":")
        lens = rng.integers(int(lo), int(hi) + 1, size=int(n))
        lens[-1] = int(hi)
    lens = np.array(lens, dtype=np.int32)
    n = len(lens)
    rows = rng.integers(1, window + 1, size=n).astype(np.int32)
    rows[0] = window
    table, blocks = wl.make_block_table(rng, lens + window, 16, spare_blocks=2)       # unused entries are -1
    d = lambda a: torch.as_tensor(a, device=DEV)
    bt, sl, nv = d(table), d(lens), d(rows) if window > 1 else None
    cand = d(wl.random_tokens(rng, n * window, SHAPE.vocab).reshape(n, window))
    kv0 = sess.kv_cache(blocks)
    kv0.normal_(generator=torch.Generator(device=DEV).manual_seed(3))
    for s in range(n):                                                                # nothing behind a context is ever read
        last = (int(lens[s]) + window + 15) // 16
        kv0[:, :, bt[s, (int(lens[s]) + 15) // 16:last].long()] = float("nan")
    max_context = int(lens.max()) + window
    ample = B.llm42_workspace_bytes(sess.model, max(n, 15), window, max_context) * 8
    ws = torch.empty(ample, dtype=torch.uint8, device=DEV)

    def run(nbytes):
        kv = kv0.clone()
        out = torch.full((n, window), -1, dtype=torch.int32, device=DEV)
        status = torch.empty(n, dtype=torch.int32, device=DEV)
        logits = torch.zeros((n, window, SHAPE.vocab), device=DEV)
        ws.fill_(0xFF)                                                                # NaN in every partial that is not written
        B.llm42_verify_window(sess.model, kv, blocks, bt, sl, cand, window, nv, max_context, out, ws[:nbytes], status, logits,
                              torch.arange(n, dtype=torch.int32, device=DEV))
        return out, status, logits, kv

    few = run(_least(lambda b: run(b), ample))
    many = run(ample)
    torch.cuda.synchronize()
    assert int(many[1].abs().max()) == 0 and torch.isfinite(many[2]).all()
    for a, b in zip(few[:3], many[:3]):
        assert torch.equal(a, b)
    assert torch.equal(few[3].view(torch.int16), many[3].view(torch.int16))           # (NaN where nothing was written)
