"""The attention kernel of decode steps and of windows of a few rows (a wave per 256-key chunk, one block of 16 query rows per
sequence and kv head) gives the same bits as the kernels of larger windows, of which the same rows are the first ones.  Those are held
to the checker in test_gpu_attention_modes.py; the schedule is fixed, so the comparison is exact.  Every case makes sure which
kernel ran: by the plan, and by the items that the call has listed in its workspace, which are chunks of 256 keys."""
import numpy as np
import pytest
import torch

from helpers import wl
from gpu_helpers import VerifierSession
from paper_2601_17768_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def sessions():
    made = {}

    def get(group):
        if group not in made:
            shape = wl.TINY.replace(d_model=512, n_q_heads=8 * group, n_kv_heads=8, head_dim=128)
            made[group] = shape, VerifierSession(shape, wl.make_weights(shape, seed=53), max_position=4608, device=DEV)
        return made[group]

    yield get
    for _, s in made.values():
        s.close()


# query heads per kv head, window, cached lengths.  Chunk and step edges: contexts of one chunk (no merge), of whole chunks, of a last
# chunk of one to four steps, past one super; sequences x 8 kv heads: fewer items than waves (1024), several per wave with
# short ones last; 4, 8, 12, 14, 15 and 16 query rows, neighbouring tokens side by side and not
CASES = [(4, 1, [0, 254, 255, 256, 257, 319, 320, 511, 512, 1023, 2000]),
         (4, 1, [2047, 63, 64, 127, 128, 191, 192, 1, 0, 300, 1279, 1280, 1281]),
         (4, 1, "uniform:0:700:60"), (4, 1, "uniform:257:300:150"), (4, 1, "uniform:0:1300:40"),
         (4, 4, [0, 251, 252, 253, 508, 1276, 2040, 2044]), (4, 4, "uniform:1:2040:40"), (4, 3, "uniform:1:2000:8"),
         (5, 3, [0, 252, 253, 254, 509, 1277, 2044, 2045]), (7, 2, "uniform:1:2040:9"), (8, 2, "uniform:1:2040:38"),
         (3, 5, [250, 251, 252, 2000, 2043, 1, 0, 700])]
# where the device decides from the lengths, and takes a wave per chunk - or not: beyond one super of sequences that deal out evenly, within
# one where a wave would get a second chunk
BY_LENGTHS = [(4, 1, [2048, 4095] + [2047, 0, 255, 256, 3000] * 3, True), (4, 1, "uniform:2100:3000:14", True), (8, 1, "uniform:1:4000:13", True),
              (4, 1, [4500] + [3, 200, 256, 257, 2048] * 5, True), (4, 2, "uniform:2060:2200:12", True), (4, 1, "uniform:3900:4094:16", False),
              (4, 1, "uniform:4000:4095:31", False), (4, 3, "uniform:3900:4090:16", False), (4, 1, [2047, 2048, 4095, 4096, 4000] * 3 + [4000], False),
              (4, 1, "uniform:0:2000:20", True), (4, 2, [2045, 2046, 0, 255, 256, 700] * 3, True), (4, 1, [1279] * 25 + [1280], False),
              (4, 1, [1280] + [1279] * 23 + [0], True), (4, 1, "uniform:1700:2040:27", False), (7, 1, [1300, 254, 255, 256] * 7, True)]


ALL = [(*c, None) for c in CASES] + BY_LENGTHS


@pytest.mark.parametrize("group,window,lens,takes", ALL, ids=[f"{g}-{w}-{c}"[:70] for g, w, c, _ in ALL])
def test_same_bits_as_the_first_rows_of_a_larger_window(sessions, group, window, lens, takes):
    shape, sess = sessions(group)
    rng = wl.rng_for(53, group, window, len(lens))
    if isinstance(lens, str):
        _, lo, hi, n = lens.split(":")
        lens = rng.integers(int(lo), int(hi) + 1, size=int(n))
        lens[-1] = int(hi)
    lens = np.array(lens, dtype=np.int32)
    n, larger = len(lens), 16 // group + 1                                            # two blocks of query rows
    rows = rng.integers(1, window + 1, size=n).astype(np.int32)
    rows[0] = window
    table, blocks = wl.make_block_table(rng, lens + larger, 16, spare_blocks=2)       # unused entries are -1
    d = lambda a: torch.as_tensor(a, device=DEV)
    bt, sl, nv = d(table), d(lens), d(rows)
    cand = d(wl.random_tokens(rng, n * larger, shape.vocab).reshape(n, larger))
    kv0 = sess.kv_cache(blocks)
    kv0.normal_(generator=torch.Generator(device=DEV).manual_seed(3))
    for s in range(n):                                                                # nothing behind a context is ever read
        last = (int(lens[s]) + larger + 15) // 16
        kv0[:, :, bt[s, (int(lens[s]) + 15) // 16:last].long()] = float("nan")

    def run(w, counts):
        max_context = int(lens.max()) + w
        plan = B.llm42_measure_attention_plan(sess.model, n, w, max_context)
        ws = torch.full((B.llm42_workspace_bytes(sess.model, n, w, max_context),), 0xFF, dtype=torch.uint8, device=DEV)   # NaN partials
        kv, out = kv0.clone(), torch.full((n, w), -1, dtype=torch.int32, device=DEV)
        status = torch.empty(n, dtype=torch.int32, device=DEV)
        logits = torch.zeros((n, w, shape.vocab), device=DEV)
        B.llm42_verify_window(sess.model, kv, blocks, bt, sl, cand[:, :w].contiguous(), w, counts, max_context, out, ws, status, logits,
                              torch.arange(n, dtype=torch.int32, device=DEV))
        torch.cuda.synchronize()
        # the items' count, a counter per layer, and the flag whose place the plan names
        control = ws[plan["sequences_flag_offset"] - 4 * (1 + shape.n_layers):plan["sequences_flag_offset"] + 4].view(torch.int32)
        return plan, (int(control[0]), int(control[-1])), out, status, logits, kv

    plan, (listed, flag), out, status, logits, kv = run(window, nv if window > 1 else None)
    assert plan["waves"] == (takes is None) and plan["may_take_waves"] == (takes is not None)
    unit = 2048 if takes is False else 256
    assert flag == int(takes is True)
    assert listed == int(((lens + rows + unit - 1) // unit).sum()) or (takes is False and int(lens.max()) + window <= 2048)   # (no list)
    ref = run(larger, nv)
    assert not ref[0]["waves"] and not ref[0]["may_take_waves"]
    assert int(status.abs().max()) == 0 and torch.isfinite(logits).all()
    assert torch.equal(out, ref[2][:, :window]) and torch.equal(status, ref[3])
    assert torch.equal(logits, ref[4][:, :window])                                    # (rows that are not there stay as they were)
    assert torch.equal(kv.view(torch.int16), ref[5].view(torch.int16))                # (NaN where nothing was written)


# sequences, window, longest context: 4 query rows per token and kv head, 8 kv heads; measured to be slower with a wave per chunk, to be
# faster, or to depend on the lengths
SLOWER = [(32, 1, 2041), (24, 1, 1001), (32, 4, 1901), (8, 1, 1001), (16, 1, 1001), (2, 1, 1901), (1, 1, 8001), (4, 1, 3001),
          (80, 1, 4501), (128, 1, 8001), (128, 1, 1901), (64, 3, 1902), (64, 4, 1004), (128, 4, 8004), (32, 4, 3004), (24, 1, 1271), (16, 4, 2044)]
FASTER = [(40, 1, 501), (48, 1, 1874), (64, 1, 1001), (8, 1, 1901), (2, 1, 1271), (16, 1, 2041), (40, 2, 1902), (40, 4, 1404), (8, 4, 1904),
          (128, 1, 1001)]
EITHER = [(24, 1, 1500), (20, 1, 1700), (28, 1, 1281), (24, 2, 1902), (16, 1, 4001), (24, 1, 3001), (64, 1, 8001), (32, 2, 2100), (16, 4, 4004)]


@pytest.mark.parametrize("n,window,max_context,how", [(*c, "no") for c in SLOWER] + [(*c, "waves") for c in FASTER] +
                         [(*c, "may_take_waves") for c in EITHER])
def test_a_wave_per_chunk_only_where_it_is_not_slower(sessions, n, window, max_context, how):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("measured with 256 CUs")
    shape, sess = sessions(4)
    plan = B.llm42_measure_attention_plan(sess.model, n, window, max_context)
    assert plan["waves"] == (how == "waves") and plan["may_take_waves"] == (how == "may_take_waves")


@pytest.mark.parametrize("n,longest", [(16, 4090), (20, 2040)])
def test_a_captured_call_chooses_at_every_replay(sessions, n, longest):
    """One captured call, replayed behind other lengths: the device takes a wave per chunk for some and not for others."""
    shape, sess = sessions(4)
    rng = wl.rng_for(53, n, longest)
    max_context = longest + 1
    table, blocks = wl.make_block_table(rng, np.full(n, max_context), 16, spare_blocks=1)
    d = lambda a: torch.as_tensor(a, device=DEV)
    bt, cand = d(table), d(wl.random_tokens(rng, n, shape.vocab).reshape(n, 1))
    kv = sess.kv_cache(blocks)
    kv.normal_(generator=torch.Generator(device=DEV).manual_seed(8))
    plan = B.llm42_measure_attention_plan(sess.model, n, 1, max_context)
    assert plan["may_take_waves"]
    ws = torch.empty(B.llm42_workspace_bytes(sess.model, n, 1, max_context), dtype=torch.uint8, device=DEV)
    sl, all_ = torch.zeros(n, dtype=torch.int32, device=DEV), torch.arange(n, dtype=torch.int32, device=DEV)
    out, logits = torch.empty((n, 1), dtype=torch.int32, device=DEV), torch.zeros((n, 1, shape.vocab), device=DEV)

    def call():
        B.llm42_verify_window(sess.model, kv, blocks, bt, sl, cand, 1, None, max_context, out, ws, None, logits, all_)

    uneven = np.concatenate([[longest], rng.integers(0, longest // 3, size=n - 1)])
    sets = [(uneven, 1), (np.full(n, longest), 0), (uneven // 2, 1), (np.full(n, longest - 7), 0), (uneven, 1)]
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for lens, waves in sets:
        sl.copy_(d(lens.astype(np.int32)))
        graph.replay()
        torch.cuda.synchronize()
        flag = ws[plan["sequences_flag_offset"]:plan["sequences_flag_offset"] + 4].view(torch.int32)
        assert int(flag[0]) == waves
        got = out.clone(), logits.clone()
        call()
        torch.cuda.synchronize()
        assert torch.isfinite(logits).all() and torch.equal(out, got[0]) and torch.equal(logits, got[1])
