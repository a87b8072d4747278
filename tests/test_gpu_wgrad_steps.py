"""The weight-gradient product at the row counts where its pipeline can go wrong: around its steps of 32 rows, its four
stages and the change from the loop without clamped loads to the one with them; odd numbers of steps, outputs that fill
neither a 256 x 256 tile nor a wave tile.  Every element against the float64 product of the stored operands (bar derived
in test_gpu_ffn_backward), routed (gathered rows) and shared, and accumulated."""
import dataclasses

import numpy as np
import pytest

from inputs import workloads as wl
from tests.helpers import require_gpu, say, to_dev
from tests.test_gpu_ffn_backward import _check_weight_grads_on_stored_operands, _forward_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 31, 32, 33, 64, 97, 128, 129, 159, 160, 161, 192, 193, 224, 255, 288, 417])
@pytest.mark.parametrize("d,f", [(128, 192), (320, 64)])
def test_rows_around_the_steps(T, d, f):
    say(f"weight gradients of {T} rows, d={d} f={f}")
    dev = require_gpu()
    E, S, k, D = 4, 1, 4, 2   # k = E: every expert has all T rows
    shape = wl.LayerShape("wgrad", T=T, d=d, f=f, E=E, S=S, k=k, D=D, dtype="bf16", components=4)
    wk = wl.make_workload(shape, seed=T)
    dy = wl.round_to_bf16(np.random.default_rng(T).standard_normal((T, d)).astype(np.float32))
    layer, _, _ = _forward_backward(shape, wk, wl.random_placement(E, D, seed=T), dy)
    _check_weight_grads_on_stored_operands(layer, shape, wk.x, dy, range(E))
    once = [g.clone() for g in (layer.dw_gate, layer.dw_up, layer.dw_down)]
    layer.expert_ffn_backward_weights(to_dev(wk.x, "bf16", dev), to_dev(dy, "bf16", dev), accumulate=True)
    for g, o in zip((layer.dw_gate, layer.dw_up, layer.dw_down), once):
        assert (g == 2 * o).all()


@pytest.mark.parametrize("T,d,f,E,S,k,skew", [
    (3200, 320, 192, 64, 1, 4, 3.0),     # 256 x 256 tiles, groups from none to hundreds of rows; both problems in one launch
    (2100, 192, 320, 128, 0, 16, 2.0),   # the same without shared experts
    (3100, 320, 192, 64, 1, 4, 0.0),     # just below the line: 128 x 128 tiles, about 200 rows in every group
    (2500, 384, 192, 6, 2, 1, 4.0),      # 128 x 128 tiles for want of larger ones; a group of more than 1024 rows
    (1100, 128, 192, 9, 1, 2, 8.0),      # the same, gathered indices fetched twice
])
def test_groups_of_all_lengths(T, d, f, E, S, k, skew):
    """Both tile sizes on batches whose groups differ (an expert's logit bias falls with its index)."""
    say(f"weight gradients T={T} d={d} f={f} E={E} S={S} k={k} skew={skew}")
    dev = require_gpu()
    shape = wl.LayerShape("wgrad", T=T, d=d, f=f, E=E, S=S, k=k, D=1, dtype="bf16", components=4)
    wk = wl.make_workload(shape, seed=T)
    bias = skew * np.linspace(1.0, 0.0, E, dtype=np.float32) * wk.logits.std()
    wk = dataclasses.replace(wk, logits=np.ascontiguousarray(wk.logits + bias, dtype=np.float32))
    dy = wl.round_to_bf16(np.random.default_rng(T).standard_normal((T, d)).astype(np.float32))
    layer, _, _ = _forward_backward(shape, wk, None, dy)
    say(f"rows per group {sorted(layer.tables()['exp_count'].tolist())}")
    _check_weight_grads_on_stored_operands(layer, shape, wk.x, dy, range(E))
    once = [g.clone() for g in (layer.dw_gate, layer.dw_up, layer.dw_down)]
    layer.expert_ffn_backward_weights(to_dev(wk.x, "bf16", dev), to_dev(dy, "bf16", dev), accumulate=True)
    for g, o in zip((layer.dw_gate, layer.dw_up, layer.dw_down), once):
        assert (g == 2 * o).all()
