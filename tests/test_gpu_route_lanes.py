"""Routing with a wavefront per token (up to 1024 tokens) and with sixteen lanes per token, and the score Gram matrix in tiles of 16 x 16, at the expert and token counts
where their lanes, registers and slices end."""
import numpy as np
import pytest
import torch

from inputs import workloads as wl
from oracle import routing
from paper_2505_13345_amd import binding as B
from paper_2505_13345_amd.layer import OccultLayer
from tests.helpers import require_gpu, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E", [1, 2, 15, 16, 17, 31, 33, 63, 65, 127, 129, 255, 256])
@pytest.mark.parametrize("k", [1, 16, 17, 32])
@pytest.mark.parametrize("T", [19, 1024, 1025])
def test_route_at_lane_edges(E, k, T):
    k = min(k, E)
    say(f"route E={E} k={k} T={T}")
    dev = require_gpu()
    lg = wl.random_logits(T, E, seed=E, scale=1.3)
    lg[::3] = np.round(lg[::3])   # ties
    ids_ref, w_ref = routing.route(lg, k, 1)
    layer = OccultLayer(T, 64, 64, E, 0, k, 1, "bf16", with_ffn=False)
    layer.route(torch.from_numpy(lg).to(dev))
    assert np.array_equal(layer.ids.cpu().numpy(), ids_ref)
    assert np.max(np.abs(layer.w.cpu().numpy().astype(np.float64) - w_ref) / w_ref) <= 1e-5   # as in test_gpu_route_plan


@pytest.mark.parametrize("E", [1, 15, 17, 60, 65, 200])
@pytest.mark.parametrize("T", [1, 3, 63, 65, 1000, 33333])
def test_gram_at_slice_edges(E, T):
    say(f"gram E={E} T={T}")
    dev = require_gpu()
    lg = wl.random_logits(T, E, seed=T, scale=1.0)
    gram = torch.full((E, E), 9.0, dtype=torch.float64, device=dev)
    B.occult_similarity_gram(B.make_cfg(T, 64, 64, E, 0, 1, 1, "bf16"), torch.from_numpy(lg).to(dev), gram)
    want = routing.gram(lg)
    got = gram.cpu().numpy()
    assert np.max(np.abs(got - want)) <= 1e-11 * np.max(np.abs(want))   # T sums of doubles: T * 2^-53 < 1e-11


@pytest.mark.parametrize("E", [7, 16, 24, 32, 60, 64, 100, 128, 200, 256])
@pytest.mark.parametrize("k", [2, 16, 20, 32])
@pytest.mark.parametrize("renorm", [0, 1])
def test_gates_do_not_depend_on_the_batch_size(E, k, renorm):
    """A token's gates are the same bits whether sixteen lanes or a wavefront route it: their sums run in one order."""
    k = min(k, E)
    say(f"gates E={E} k={k} renorm={renorm}")
    dev = require_gpu()
    T, part = 1500, 700
    lg = torch.from_numpy(wl.random_logits(T, E, seed=E + k, scale=1.7)).to(dev)
    large, small = (OccultLayer(n, 64, 64, E, 0, k, 1, "bf16", 0, 1, renorm, with_ffn=False) for n in (T, part))
    large.route(lg)
    small.route(lg[:part].contiguous())
    assert torch.equal(large.ids[:part], small.ids)
    assert torch.equal(large.w[:part].view(torch.int32), small.w.view(torch.int32))
