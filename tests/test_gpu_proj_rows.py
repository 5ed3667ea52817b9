"""Decoder parity at the row counts where the projections change kernel: the
edges of four to eight 16-row tiles (128 rows is the most the split-K kernel
takes), and slices longer than its ring."""
import numpy as np
import pytest

from pced_inputs import workloads as W
from pced_inputs.model import ModelSpec

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [49, 64, 65, 80, 81, 97, 113, 128, 129])
def test_row_tiles(rows):
    from tests.test_gpu_model import _run
    geom = W.Geometry(2, 4, 2, 64, 256, 300, "bf16")
    wl = W.custom(geom, [rows - 1], np.random.default_rng(rows).integers(1, 40, size=rows - 1).tolist(), amateur_len=5,
                  steps=1, seed=rows)
    assert _run(wl, ModelSpec(geom, ffn_dim=1408, rope_theta=10000.0, seed=rows), steps=1) <= 1


@pytest.mark.parametrize("experts,prefill", [([2], 0), ([32], 0), ([69], 0), ([2], 22)])
def test_long_slices(experts, prefill):
    """Hidden 2048: K slices of 16 steps; a prefill chunk of 66 rows."""
    from tests.test_gpu_model import _run
    geom = W.Geometry(1, 16, 4, 128, 2048, 300, "bf16")
    n = sum(experts)
    wl = W.custom(geom, experts, np.random.default_rng(n).integers(1, 40, size=n).tolist(), amateur_len=5, steps=1,
                  seed=n)
    _run(wl, ModelSpec(geom, ffn_dim=5632, rope_theta=10000.0, seed=n), steps=1, prefill=prefill)
