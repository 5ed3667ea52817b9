"""The fp32 kernels at the edges of their tiles, against float64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("rows,vocab,hq,d", [
    (1, 2, 1, 4),         # less than one unit of the hidden dimension, one partial vocab tile
    (16, 17, 1, 36), (17, 16, 3, 12), (5, 1000, 4, 64),
    (33, 1003, 5, 80), (48, 15, 2, 100), (49, 33, 4, 128),   # 49 rows: a second row group
    (49, 8191, 2, 20), (100, 8192, 2, 20),                  # the most with one vocab tile per block; two
    (100, 16384, 2, 20), (19, 16421, 1, 128),
])
@pytest.mark.parametrize("norm", ["rms", "none"])
def test_lmhead_f32(rows, vocab, hq, d, norm):
    from paper_2601_08670_amd import _lib
    K = hq * d
    cfg = _lib.make_config(n_layers=1, n_q_heads=hq, n_kv_heads=1, head_dim=d, vocab=vocab, dtype="f32",
                           max_queries=1, max_seqs=max(2, rows), max_pages=1, max_pages_per_seq=1, norm=norm)
    ctx = _lib.Context(cfg, device=DEV)
    g = torch.Generator().manual_seed(rows * 1000 + vocab)
    x, w = torch.randn(rows, K, generator=g), 0.02 * torch.randn(vocab, K, generator=g)
    wp = torch.empty(_lib.pced_lm_head_bytes(cfg), dtype=torch.uint8, device=DEV)
    _lib.pced_pack_lm_head(cfg, w.to(DEV), wp)
    out = torch.full((rows, vocab), float("nan"), device=DEV)
    ctx.pced_lmhead(x.to(DEV), rows, wp, out)
    x64, w64 = x.double(), w.double()
    rho = torch.rsqrt(x64.square().mean(1, keepdim=True) + 1e-5) if norm == "rms" else torch.ones(rows, 1).double()
    # K products summed in fp32 in any order, then the row scale (a sum of K squares, a square root, a division)
    bound = (2 * K + 8) * 2.0 ** -24 * (x64.abs() @ w64.abs().T) * rho
    err = (out.cpu().double() - (x64 @ w64.T) * rho).abs()
    assert np.isfinite(out.cpu().numpy()).all() and bool((err <= bound).all()), float((err / bound).max())


@pytest.mark.parametrize("hq,hkv,d,lens,chunks", [
    (1, 1, 4, [1, 16], 0), (3, 3, 12, [15, 17], 0), (16, 1, 32, [40, 100], 0), (7, 1, 36, [31, 64], 0),
    (4, 2, 64, [128, 250, 5], 0), (5, 5, 80, [33, 90], 3), (8, 4, 100, [200, 1], 1), (16, 4, 128, [16, 700], 2),
])
def test_attention_f32(hq, hkv, d, lens, chunks):
    """Two steps over caches whose reserved slots hold NaN; several pages and sequences per chunk, and split ones."""
    from paper_2601_08670_amd.session import PcedSession
    S, L, G = len(lens), 2, hq // hkv
    need = [-(-(n + 2) // 16) for n in lens]
    g = torch.Generator().manual_seed(hq * 100 + d)
    rnd = lambda *shape: torch.randn(*shape, generator=g)  # noqa: E731
    k, v = [rnd(L, n, hkv, d) for n in lens], [rnd(L, n, hkv, d) for n in lens]
    sess = PcedSession(n_layers=L, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, vocab=33, dtype="f32", max_queries=1,
                       max_seqs=S, max_pages=sum(need), max_pages_per_seq=max(need), device=DEV, poison=True,
                       max_attn_chunks=chunks)
    sess.load([S - 1], lens, [t.to(DEV) for t in k], [t.to(DEV) for t in v], [0.5] * (S - 1), reserve_tokens=2)
    w = sess.pack_lm_head(rnd(33, hq * d).to(DEV))
    eps = 2.0 ** -24
    for _ in range(2):
        q, kn, vn = rnd(S, L, hq, d), rnd(S, L, hkv, d), rnd(S, L, hkv, d)
        got = sess.step(q.to(DEV), kn.to(DEV), vn.to(DEV), w, want=("attn_out", "hidden"))
        out = got["attn_out"].cpu().double()
        for s in range(S):
            k[s] = torch.cat([k[s], kn[s][:, None]], 1)
            v[s] = torch.cat([v[s], vn[s][:, None]], 1)
            T = k[s].shape[1]
            kk, vv = (t[s].double().repeat_interleave(G, 2) for t in (k, v))  # [L][T][hq][d]
            z = torch.einsum("lhd,lthd->lht", q[s].double(), kk) / d ** 0.5
            ref = torch.einsum("lht,lthd->lhd", z.softmax(-1), vv)
            # scores: d products and their scaling; weights: the score's error, exp2, sums over T terms
            dz = (d + 8) * eps * torch.einsum("lhd,lthd->lht", q[s].double().abs(), kk.abs()).max().item() / d ** 0.5
            bound = 2 * (2 * dz + (T + 32) * eps) * vv.abs().max().item()
            assert (out[s] - ref).abs().max().item() <= bound, (s, T)
        assert torch.equal(got["hidden"].view(S, hq, d), got["attn_out"][:, -1])


def _lane_sum_f32(k):
    """Sums of rows [n][d] in fp32 by halves of a 64-wide tree (elements i and i + 64 first)."""
    t = np.zeros((len(k), 128), np.float32)
    t[:, :k.shape[1]] = k
    w = 64
    while w:
        t = t[:, :w] + t[:, w:2 * w]
        w //= 2
    return t[:, 0]


@pytest.mark.parametrize("d", [20, 64, 80, 128])
def test_attention_f32_score_rounding(d):
    """The rounding of a score's d products stays that of a tree: 16 keys whose exact scores are
    equal (orders of the same elements, sum nearly 0) and one-hot values, so that the outputs are
    the weights and their logarithms the scores' errors."""
    from paper_2601_08670_amd.session import PcedSession
    S, L, T, c = 64, 4, 16, 64.0
    g = np.random.default_rng(d)
    k = np.empty((S, L, T, d), np.float32)
    for s in range(S):
        for l in range(L):
            row = g.standard_normal(d).astype(np.float32)
            row[-1] = -row[:-1].astype(np.float64).sum()
            for t in range(T):
                k[s, l, t] = g.permutation(row)
    v = torch.eye(T, d).view(1, T, 1, d).expand(L, -1, -1, -1)
    kk = torch.from_numpy(k)
    sess = PcedSession(n_layers=L, n_q_heads=4, n_kv_heads=1, head_dim=d, vocab=17, dtype="f32", max_queries=1,
                       max_seqs=S, max_pages=S, max_pages_per_seq=1, device=DEV)
    sess.load([S - 1], [T - 1] * S, [kk[s, :, :T - 1, None].contiguous().to(DEV) for s in range(S)],
              [v[:, :T - 1].contiguous().to(DEV)] * S, [0.5] * (S - 1), reserve_tokens=1)
    q = torch.full((S, L, 4, d), c)  # (a power of two: the products are exact)
    out = sess.step(q.to(DEV), kk[:, :, T - 1:].contiguous().to(DEV), v[None, :, T - 1].expand(S, -1, -1, -1).contiguous().to(DEV),
                    sess.pack_lm_head(torch.randn(17, 4 * d).to(DEV)), want=("attn_out",))["attn_out"]
    z = np.log(out[:, :, 0, :T].cpu().double().numpy()) * d ** 0.5 / c

    def rms(x):  # about each sequence's mean: the softmax does not see a common offset
        x = x.reshape(-1, T)
        return float(np.sqrt(np.square(x - x.mean(1, keepdims=True)).mean()))

    tree = rms(_lane_sum_f32(k.reshape(-1, d)).astype(np.float64))
    # 4096 errors of each (1.6% of sampling in their ratio), a few ulp of weights near 1/16 and their logarithms
    assert rms(z) <= 1.1 * tree + 4 * 2.0 ** -24 * d ** 0.5 / c, (rms(z), tree)
