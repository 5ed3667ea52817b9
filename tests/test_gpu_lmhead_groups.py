"""The bf16 LM head over more rows than one block holds (row groups): logits
against float64, and the fused token choice against the one made from
materialised logits (the same arithmetic: equal bits)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("rows,vocab,hidden,noalloc", [
    (288, 777, 256, False),      # the largest single group
    (289, 1003, 256, False),     # two groups of 10 tiles, the last of 1 row
    (321, 4096, 512, True), (385, 17, 256, False), (449, 2300, 256, True), (576, 513, 1024, False),
    (577, 300, 256, False),      # three groups
    (1200, 2049, 256, False),
    # vocabularies of enough chunks for row groups (the ones above fit the 48-row kernel in one round)
    (289, 9700, 256, False), (289, 40, 4096, True), (321, 9500, 512, True), (385, 9001, 1024, False),
    (449, 9000, 1024, True), (576, 7003, 768, False), (577, 6000, 1024, False), (1200, 3000, 1024, False),
    (480, 8000, 256, False), (480, 16400, 256, False),   # short hidden size: two rounds of the 48-row kernel, and more
])
def test_lmhead_row_groups(rows, vocab, hidden, noalloc):
    from paper_2601_08670_amd import _lib
    cfg = _lib.make_config(n_layers=1, n_q_heads=hidden // 64, n_kv_heads=hidden // 256, head_dim=64, vocab=vocab,
                           dtype="bf16", max_queries=1, max_seqs=rows, max_pages=1, max_pages_per_seq=1)
    ctx = _lib.Context(cfg, device=DEV)
    g = torch.Generator().manual_seed(rows)
    x, w = torch.randn(rows, hidden, generator=g).bfloat16(), (0.02 * torch.randn(vocab, hidden, generator=g)).bfloat16()
    wp = torch.empty(_lib.pced_lm_head_bytes(cfg), dtype=torch.uint8, device=DEV)
    _lib.pced_pack_lm_head(cfg, w.to(DEV), wp)
    out = torch.full((rows, vocab), float("nan"), device=DEV)
    if noalloc:
        _lib.pced_lmhead_noalloc(cfg, x.to(DEV), rows, wp, out)
    else:
        ctx.pced_lmhead(x.to(DEV), rows, wp, out)
    x64, w64 = x.double(), w.double()
    rho = torch.rsqrt(x64.square().mean(1, keepdim=True) + 1e-5)
    # exact bf16 products, fp32 sums of `hidden` terms in any order, the row scale
    bound = (2 * hidden + 8) * 2.0 ** -24 * (x64.abs() @ w64.abs().T) * rho
    err = (out.cpu().double() - (x64 @ w64.T) * rho).abs()
    assert bool((err <= bound).all()), float((err / bound).max())


@pytest.mark.parametrize("experts,vocab", [
    ([90] * 4, 2048),               # two groups of two queries
    ([287, 1], 1003),               # one query fills a group
    ([70, 141, 3, 100, 30], 515),   # ragged groups
    ([1] * 150 + [13], 300),        # many queries per group
    ([288, 2], 300), ([288, 2], 9500),  # a query larger than a group: not fused
    ([90] * 4, 8300), ([287, 1], 9500), ([70, 141, 3, 100, 30], 8303), ([1] * 150 + [13], 9500),  # (row groups, as above)
])
def test_fused_choice_over_row_groups(experts, vocab):
    from paper_2601_08670_amd.session import PcedSession
    S, NE = sum(experts) + len(experts), sum(experts)
    g = torch.Generator(DEV).manual_seed(S)
    rnd = lambda *shape: torch.randn(*shape, device=DEV, generator=g).bfloat16()  # noqa: E731
    lens = [1 + i % 3 for i in range(S)]
    k, v = [rnd(1, n, 1, 64) for n in lens], [rnd(1, n, 1, 64) for n in lens]
    q, kn, vn, w = rnd(S, 1, 4, 64), rnd(S, 1, 1, 64), rnd(S, 1, 1, 64), rnd(vocab, 256)
    r = np.random.RandomState(S)
    rel, beta = r.uniform(0.05, 0.95, NE).tolist(), r.uniform(0.1, 1.0, NE).tolist()
    got = []
    for want in (("winner", "top1", "top2"), ("winner", "top1", "top2", "logits")):  # fused, materialised
        sess = PcedSession(n_layers=1, n_q_heads=4, n_kv_heads=1, head_dim=64, vocab=vocab, dtype="bf16",
                           max_queries=len(experts), max_seqs=S, max_pages=S, max_pages_per_seq=1, device=DEV,
                           poison=True)
        sess.load(experts, lens, k, v, rel, beta=beta)
        got.append(sess.step(q, kn, vn, sess.pack_lm_head(w), want=want))
    for name in ("tokens", "winner", "top1", "top2"):
        assert torch.equal(got[0][name], got[1][name]), name


@pytest.mark.parametrize("vocab", [300, 9700])  # the 48-row kernel; row groups
def test_decoder_stack_beyond_288_rows(vocab):
    """Rows whose scales come from the final norm's sums."""
    from pced_inputs import workloads as W
    from pced_inputs.model import ModelSpec
    from tests.test_gpu_model import _run
    geom = W.Geometry(1, 4, 1, 64, 256, vocab, "bf16")
    wl = W.custom(geom, [150, 148], [1 + i % 7 for i in range(298)], amateur_len=3, steps=2, seed=vocab)
    _run(wl, ModelSpec(geom, ffn_dim=128, rope_theta=10000.0, seed=vocab), steps=2)
