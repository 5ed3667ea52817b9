"""Prefill attention at the edges of its token groups: one and two 16-column
tiles, one group alone up to two blocks of groups (so 1, 2, 4 and 8 page units
per wave), ragged last groups, pages shorter than the ring and long ones split
over chunks. The second layer's K/V rows check the first layer's attention for
every suffix token."""
import pytest

from pced_inputs import workloads as W
from pced_inputs.model import ModelSpec

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d,n_tok,cap", [
    (4, 1, 128, 1, 0), (4, 1, 128, 4, 0), (4, 1, 128, 5, 0), (4, 1, 128, 8, 2),  # one group, one or two tiles
    (4, 1, 128, 9, 0), (4, 1, 128, 17, 0), (4, 1, 128, 33, 3),                   # 2, 3 and 5 groups
    (4, 1, 128, 63, 0), (4, 1, 128, 70, 2),                                      # 8 groups; 9 in two blocks
    (4, 4, 64, 32, 0), (4, 4, 64, 33, 4), (4, 4, 64, 97, 0),                     # 32 tokens per group: 1, 2 and 4 groups
    (20, 4, 64, 13, 0), (14, 2, 128, 9, 0),                                      # 5 and 7 q-heads per kv-head
])
def test_group_edges(hq, hkv, d, n_tok, cap):
    from tests.test_gpu_model import _run
    geom = W.Geometry(2, hq, hkv, d, hq * d, 500, "bf16")
    wl = W.custom(geom, [3], [1, 150, 47], amateur_len=16, steps=1, seed=n_tok)
    _run(wl, ModelSpec(geom, ffn_dim=512, rope_theta=10000.0, seed=n_tok), steps=1, prefill=n_tok,
         max_attn_chunks=cap)


@pytest.mark.parametrize("hq,hkv,d,n_tok,cap", [(4, 1, 128, 9, 1), (4, 1, 128, 40, 1), (4, 4, 64, 3, 2)])
def test_chunk_over_many_short_sequences(hq, hkv, d, n_tok, cap):
    # chunks of about 50 pages: one holds some 30 of the short caches and the start of the long one
    from tests.test_gpu_model import _run
    geom = W.Geometry(2, hq, hkv, d, hq * d, 500, "bf16")
    wl = W.custom(geom, [32], [3 + i % 9 for i in range(30)] + [1100, 5], amateur_len=16, steps=1, seed=n_tok)
    _run(wl, ModelSpec(geom, ffn_dim=512, rope_theta=10000.0, seed=n_tok), steps=1, prefill=n_tok,
         max_attn_chunks=cap)
