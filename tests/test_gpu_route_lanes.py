"""Routing with a wavefront per token (up to 1024 tokens) and with sixteen lanes per token, and the score Gram matrix in
tiles of 16 x 16, at the expert and token counts where their lanes, registers and slices end."""
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


PRUNE_CASES = [
    # E, D, k, n_d: experts, devices and slots per lane of sixteen
    (8, 8, 3, 3),        # fewer experts than lanes
    (16, 4, 4, 2),
    (32, 4, 17, 3),      # two experts per lane, slots in both registers
    (32, 16, 4, 3),
    (48, 24, 20, 12),    # two registers of devices, the second half filled
    (64, 32, 4, 3),
    (64, 64, 17, 20),    # four registers of devices
    (64, 64, 32, 40),
    (128, 32, 16, 4),
    (256, 4, 32, 1),
    (256, 64, 17, 9),
]


@pytest.mark.parametrize("T", [900, 1026, 2051])   # a wavefront per token; sixteen lanes, the last wave half empty
@pytest.mark.parametrize("mode", [1, 2, 3])
@pytest.mark.parametrize("E,D,k,n_d", PRUNE_CASES)
def test_pruned_route_at_lane_edges(E, D, k, n_d, mode, T):
    say(f"pruned route E={E} D={D} k={k} n_d={n_d} mode={mode} T={T}")
    dev = require_gpu()
    lg = wl.random_logits(T, E, seed=E + D + k, scale=1.3)
    lg[::3] = np.round(lg[::3])   # ties
    pos = wl.random_placement(E, D, seed=E + D)
    tab = routing.similarity_table(routing.gram(wl.random_logits(500, E, seed=k, scale=1.0))) if mode == 3 else None
    ids_ref, w_ref = routing.route(lg, k, D, pos, n_d=n_d, prune_mode=mode, renorm=1, sim_table=tab)
    layer = OccultLayer(T, 64, 64, E, 0, k, D, "bf16", n_d, mode, 1, pos, with_ffn=False, sim_table=tab)
    layer.route(torch.from_numpy(lg).to(dev))
    assert np.array_equal(layer.ids.cpu().numpy(), ids_ref)
    assert np.max(np.abs(layer.w.cpu().numpy().astype(np.float64) - w_ref) / w_ref) <= 1e-5   # as in test_gpu_route_plan


@pytest.mark.parametrize("E,D,k,n_d,mode", [(16, 4, 4, 0, 1), (64, 8, 8, 2, 1), (60, 4, 4, 2, 2), (32, 4, 17, 3, 3),
                                            (256, 16, 8, 4, 1)])
def test_non_finite_scores_with_sixteen_lanes(E, D, k, n_d, mode):
    """NaN, -inf and +inf scores in a batch of more than 1024 tokens: k distinct experts in range on n_d devices, finite gates,
    and the tokens beside them in their wavefront routed as the oracle routes them."""
    say(f"non-finite scores E={E} D={D} k={k} n_d={n_d} mode={mode}")
    dev = require_gpu()
    T = 1300
    lg = wl.random_logits(T, E, seed=E + k, scale=1.3)
    tab = routing.similarity_table(routing.gram(lg[:500])) if mode == 3 else None
    rng = np.random.default_rng(E)
    bad = rng.choice(T, size=260, replace=False)
    for i, t in enumerate(bad):
        lg[t, rng.choice(E, size=[1, E // 2, E - 1, E][i % 4], replace=False)] = [np.nan, -np.inf, np.inf][i % 3]
    layer = OccultLayer(T, 64, 64, E, 0, k, D, "bf16", n_d, mode, 1, with_ffn=False, sim_table=tab)
    layer.route(torch.from_numpy(lg).to(dev))
    ids, w = layer.ids.cpu().numpy(), layer.w.cpu().numpy()
    good = np.setdiff1d(np.arange(T), bad)
    ids_ref, w_ref = routing.route(lg[good], k, D, n_d=n_d, prune_mode=mode, renorm=1, sim_table=tab)
    assert np.array_equal(ids[good], ids_ref)
    assert np.max(np.abs(w[good] - w_ref) / w_ref) <= 1e-5
    assert ids.min() >= 0 and ids.max() < E and np.isfinite(w).all()
    assert all(len(set(row)) == k for row in ids.tolist())
    if n_d:
        assert all(len({e // (E // D) for e in row}) <= n_d for row in ids.tolist())
