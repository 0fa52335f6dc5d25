"""Attention by chunks of 256 keys at head dimension 128: which calls of 8 and more blocks of query rows run it with 4 waves and two
workgroups to a CU instead of 8 waves and one."""
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
