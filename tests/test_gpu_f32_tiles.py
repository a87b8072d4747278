"""The float32 expert products (32 x 64 tiles, K tiles of 64) at the sizes where they can go wrong: rows around a row tile,
column tiles cut by N, K below, at and just above a K tile, empty groups, a shared down projection whose K walks matrices
narrower than a K tile, more than 64 groups.  Every stored tensor against the float64 product of its own stored operands."""
import numpy as np
import pytest
import torch

from inputs import workloads as wl
from paper_2505_13345_amd.layer import OccultLayer
from tests.helpers import require_gpu, say, to_dev

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def product(a, b):
    """a b^T and the bound on any order of f32 sums of it: K products, K sums, each within U of its value."""
    return a @ b.T, 1.01 * (a.shape[1] + 1) * U * (np.abs(a) @ np.abs(b).T)


def check(got, ref, bound, what):
    worst = np.max(np.abs(got - ref) - bound - 1e-37)
    assert worst <= 0.0, f"{what}: {worst:.3e} beyond the bound"


@pytest.mark.parametrize("T,d,f,E,S,k,D", [
    (32, 64, 64, 4, 0, 4, 2),       # one whole row tile per expert, one K tile, one column tile
    (33, 68, 60, 4, 1, 4, 2),       # one row more; a K tile of 4; columns cut
    (31, 4, 12, 2, 3, 2, 1),        # the shortest K; shared K of 3 matrices of 12
    (65, 128, 100, 3, 2, 2, 3),     # two whole K tiles; up half cut inside a tile
    (9, 192, 196, 70, 1, 1, 7),     # more than 64 groups, most of them empty
    (500, 256, 320, 2, 1, 1, 2),    # hundreds of rows, five K tiles
])
def test_f32_products(T, d, f, E, S, k, D):
    say(f"f32 tiles T={T} d={d} f={f} E={E} S={S} k={k}")
    dev = require_gpu()
    wk = wl.make_workload(wl.LayerShape("f32t", T=T, d=d, f=f, E=E, S=S, k=k, D=D, dtype="f32", components=4), seed=T + d)
    layer = OccultLayer(T, d, f, E, S, k, D, "f32")
    x = to_dev(wk.x, "f32", dev)
    w = [to_dev(a, "f32", dev) for a in (wk.w_gate, wk.w_up, wk.w_down)]
    layer.forward(torch.from_numpy(wk.logits).to(dev), x, *w, train=True)
    torch.cuda.synchronize()
    f64 = lambda t: t.double().cpu().numpy()
    tab = layer.tables()
    off, expert, src = (tab[n].cpu().numpy() for n in ("exp_offset", "pos_expert", "epd_sfd_row"))
    sfd_x, gu, h, y = (f64(t) for t in (layer.sfd_x, layer.epd_gu, layer.epd_h, layer.epd_y))
    W = [np.asarray(a, dtype=np.float64) for a in (wk.w_gate, wk.w_up, wk.w_down)]

    def first(tag, e, rows_x, rows_gu, rows_h):
        (g, dg), (u, du) = product(rows_x, W[0][e]), product(rows_x, W[1][e])
        check(rows_gu, np.concatenate([g, u], 1), np.concatenate([dg, du], 1), f"pre-activations {tag}")
        silu = g / (1.0 + np.exp(-g))   # |silu'| <= 1.1; exp, sum, quotient and product each round (16 U covers expf too)
        check(rows_h, silu * u, 1.1 * dg * (np.abs(u) + du) + np.abs(silu) * du + 16 * U * np.abs(silu * u), f"h {tag}")

    for P in range(E):
        r, e = slice(off[P], off[P + 1]), int(expert[P])
        if off[P + 1] > off[P]:
            first(f"expert {e}", e, sfd_x[src[r]], gu[r], h[r])
            check(y[r], *product(h[r], W[2][e]), f"y expert {e}")
    if S:
        hs, gs = f64(layer.h_shared), f64(layer.gu_shared)
        for s in range(S):
            first(f"shared {s}", E + s, wk.x.astype(np.float64), gs[:, 2 * s * f:2 * (s + 1) * f], hs[:, s * f:(s + 1) * f])
        check(f64(layer.y_shared), *product(hs, np.concatenate([W[2][E + s] for s in range(S)], axis=1)), "y shared")
