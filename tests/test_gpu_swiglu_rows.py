"""Gate/up in one K slice (hidden 256), with its epilogue in the projection launch at
the row-tile edges up to 48 rows (more: test_gpu_proj_rows.py), and as two launches
where the columns give more blocks than compute units; the activations are compared
stage-wise."""
import numpy as np
import pytest

from pced_inputs import workloads as W
from pced_inputs.model import ModelSpec

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,ffn", [(2, 64), (16, 1408), (17, 64), (33, 1408), (48, 192), (5, 16384), (17, 16448)])
def test_swiglu_rows(rows, ffn):
    from tests.test_gpu_model import _run
    geom = W.Geometry(2, 4, 2, 64, 256, 300, "bf16")
    wl = W.custom(geom, [rows - 1], np.random.default_rng(rows).integers(1, 40, size=rows - 1).tolist(), amateur_len=5,
                  steps=1, seed=rows)
    assert _run(wl, ModelSpec(geom, ffn_dim=ffn, rope_theta=10000.0, seed=rows), steps=1) <= 1
