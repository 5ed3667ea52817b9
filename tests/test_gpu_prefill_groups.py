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


@pytest.mark.parametrize("hq,hkv,d,n_tok,bad", [
    (4, 1, 128, 16, 8), (4, 1, 128, 16, 4), (4, 1, 128, 40, 23), (4, 4, 64, 40, 16), (4, 4, 64, 70, 65),
])
def test_later_tokens_leave_earlier_ones_alone(hq, hkv, d, n_tok, bad):
    """A suffix token whose embedding is NaN (so that all of its K and V rows are): tokens before
    the 16-column tile that it falls in get the bits they get beside an ordinary token."""
    from paper_2601_08670_amd.session import PcedSession
    g = torch.Generator().manual_seed(n_tok)
    L, H, F, V, lens = 2, hq * d, 256, 500, [20, 3, 150]
    rnd = lambda *shape, s=1.0: (s * torch.randn(*shape, generator=g)).bfloat16().to("cuda:0")  # noqa: E731
    sess = PcedSession(n_layers=L, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, vocab=V, dtype="bf16", max_queries=1,
                       max_seqs=3, max_pages=60, max_pages_per_seq=20, ffn_dim=F)
    k, v = [rnd(L, n, hkv, d) for n in lens], [rnd(L, n, hkv, d) for n in lens]
    shapes = [(H,), (H, H), (hkv * d, H), (hkv * d, H), (H, H), (H,), (F, H), (F, H), (H, F)]
    layers = [[rnd(*s, s=0.05) if len(s) > 1 else rnd(*s) for s in shapes] for _ in range(L)]
    embed = rnd(V, H)
    embed[V - 1] = float("nan")
    model = sess.pack_model(lambda l: layers[l], embed, rnd(H))
    tokens = torch.randint(0, V - 1, (1, n_tok), generator=g, dtype=torch.int32).to("cuda:0")
    got = []
    for t in (int(tokens[0, bad]), V - 1):
        tokens[0, bad] = t
        sess.load([2], lens, k, v, [0.5, 0.5], reserve_tokens=n_tok)
        sess.ctx.pced_model_prefill(model, n_tokens=n_tok, tokens=tokens)
        got.append([sess.read_cache(s, L - 1, n, n_tok) for s, n in enumerate(lens)])
    gk = hq // hkv
    sure = bad * gk // 16 * 16 // gk  # tokens whose columns all lie in earlier tiles
    assert 0 < sure <= bad
    for (k0, v0), (k1, v1) in zip(*got):
        assert torch.equal(k0[:sure], k1[:sure]) and torch.equal(v0[:sure], v1[:sure])
        nan = v1[bad].view(torch.bfloat16).float().isnan()
        assert bool(nan.all()) and bool(v0.view(torch.bfloat16).float().isfinite().all())
