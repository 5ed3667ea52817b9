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
    (100, 16384, 2, 20), (19, 16421, 1, 128),               # two vocab tiles per block
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
