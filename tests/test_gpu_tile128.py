"""The 128-row tiles of the grouped expert products (routed and shared experts in one launch), at the sizes where they
can go wrong: rows around a tile, half-filled column tiles, the shortest K (three and four K tiles), more than 64 groups,
empty groups, a shared down projection whose K walks several matrices.  Every stored tensor against the float64
product of its own stored operands, element by element."""
import numpy as np
import pytest
import torch

from inputs import workloads as wl
from paper_2505_13345_amd import binding as B
from paper_2505_13345_amd.layer import OccultLayer
from tests.helpers import assert_one_rounding, require_gpu, say, to_dev

pytestmark = pytest.mark.gpu

CASES = [
    # T, d, f, E, S, k, D
    (128, 192, 192, 4, 1, 4, 2),      # exactly one row tile per expert (k = E), three K tiles everywhere
    (129, 192, 320, 4, 2, 4, 2),      # one row more; half-filled column tiles; shared K of 2 x 320
    (127, 256, 448, 2, 3, 2, 1),      # one row less; four K tiles
    (640, 320, 192, 132, 1, 4, 2),    # more than 64 groups, a few rows each
    (300, 192, 256, 96, 1, 1, 4),     # some groups empty
    (900, 512, 704, 8, 0, 2, 4),      # no shared experts; two row tiles per group
    (700, 1088, 192, 12, 1, 4, 3),    # column tiles of 1088 outputs: 4 whole and a quarter
]


@pytest.mark.parametrize("T,d,f,E,S,k,D", CASES)
def test_tile128_products(T, d, f, E, S, k, D, logits=None):
    say(f"128-row tiles T={T} d={d} f={f} E={E} S={S} k={k}")
    dev = require_gpu()
    wk = wl.make_workload(wl.LayerShape("t128", T=T, d=d, f=f, E=E, S=S, k=k, D=D, dtype="bf16", components=4), seed=T + d)
    layer = OccultLayer(T, d, f, E, S, k, D, "bf16")
    x = to_dev(wk.x, "bf16", dev)
    wg, wu, wd = (to_dev(a, "bf16", dev) for a in (wk.w_gate, wk.w_up, wk.w_down))
    layer.forward(torch.from_numpy(wk.logits if logits is None else logits).to(dev), x, wg, wu, wd, train=True)
    layer.transpose_weights(wg, wu, wd)
    dy = wl.round_to_bf16(np.random.default_rng(T).standard_normal((T, d)).astype(np.float32))
    _, epd_dy, _ = layer.combine_backward(to_dev(dy, "bf16", dev))
    gu_fwd = layer.epd_gu.double().cpu().numpy()
    gu_sh_fwd = layer.gu_shared.double().cpu().numpy() if S else None
    layer.expert_ffn_backward(x, wg, wu, epd_dy, to_dev(dy, "bf16", dev))
    torch.cuda.synchronize()
    f64 = lambda t: t.double().cpu().numpy()
    tab = layer.tables()
    off, expert = tab["exp_offset"].cpu().numpy(), tab["pos_expert"].cpu().numpy()
    src = tab["epd_sfd_row"].cpu().numpy()
    sfd_x, h, y, dh, dgu, dx, dyq = (f64(t) for t in (layer.sfd_x, layer.epd_h, layer.epd_y, layer.epd_dh, layer.epd_gu,
                                                     layer.epd_dx, epd_dy))
    W = [np.asarray(a, dtype=np.float64) for a in (wk.w_gate, wk.w_up, wk.w_down)]

    def check(tag, e, rows_x, rows_gu, rows_h, rows_dy, rows_dh):
        g, u = rows_x @ W[0][e].T, rows_x @ W[1][e].T
        assert_one_rounding(rows_gu, np.concatenate([g, u], axis=1), f"pre-activations {tag}")
        assert_one_rounding(rows_h, g / (1.0 + np.exp(-g)) * u, f"h {tag}")
        assert_one_rounding(rows_dh, rows_dy @ W[2][e], f"dh {tag}")

    for P in range(E):
        r = slice(off[P], off[P + 1])
        if off[P + 1] == off[P]:
            continue
        e = int(expert[P])
        check(f"expert {e}", e, sfd_x[src[r]], gu_fwd[r], h[r], dyq[r], dh[r])
        assert_one_rounding(y[r], h[r] @ W[2][e].T, f"y expert {e}")
        assert_one_rounding(dx[r], dgu[r, :f] @ W[0][e] + dgu[r, f:] @ W[1][e], f"dx expert {e}")
    if S:
        hs, ys, dhs, dgus, dxs = (f64(t) for t in (layer.h_shared, layer.y_shared, layer.dh_shared, layer.gu_shared,
                                                   layer.dx_shared))
        y_ref, dx_ref = np.zeros((T, d)), np.zeros((T, d))
        for s in range(S):
            c, c2 = slice(s * f, (s + 1) * f), slice(s * 2 * f, (s + 1) * 2 * f)
            check(f"shared {s}", E + s, wk.x.astype(np.float64), gu_sh_fwd[:, c2], hs[:, c], dy.astype(np.float64), dhs[:, c])
            y_ref += hs[:, c] @ W[2][E + s].T
            dx_ref += dgus[:, c2][:, :f] @ W[0][E + s] + dgus[:, c2][:, f:] @ W[1][E + s]
        assert_one_rounding(ys, y_ref, "y shared")
        assert_one_rounding(dxs, dx_ref, "dx shared")


def test_activation_of_groups_of_a_few_rows_divides_first():
    """50 routed rows per group and 100 shared ones: silu(g) * u is g / (1 + exp(-g)) first, with the f32 division, and
    then times u, so a large negative gate beside a large up value gives -0 (g * u alone overflows f32); the other
    values are the f64 activation rounded once."""
    T, d, f, E, S, k, D = 100, 192, 192, 4, 1, 2, 2
    say(f"activation T={T} E={E} S={S} k={k}")
    dev = require_gpu()
    wk = wl.make_workload(wl.LayerShape("silu", T=T, d=d, f=f, E=E, S=S, k=k, D=D, dtype="bf16", components=4), seed=3)
    x, wg, wu = wk.x.copy(), wk.w_gate.copy(), wk.w_up.copy()
    wg[:, :32, 0], wu[:, :32, 0] = -2.0 ** 33, 2.0 ** 33
    x[::3] = 0.0
    x[::3, 0] = 2.0 ** 33          # gate -2^66, up 2^66 in the first 32 columns of these tokens
    x[1::3, 0] = x[2::3, 0] = 0.0
    layer = OccultLayer(T, d, f, E, S, k, D, "bf16")
    layer.forward(torch.from_numpy(wk.logits).to(dev), *(to_dev(a, "bf16", dev) for a in (x, wg, wu, wk.w_down)))
    torch.cuda.synchronize()
    tab = layer.tables()
    off, expert = tab["exp_offset"].cpu().numpy(), tab["pos_expert"].cpu().numpy()
    src = tab["epd_sfd_row"].cpu().numpy()
    sfd_x = layer.sfd_x.double().cpu().numpy()
    groups = [(int(expert[P]), sfd_x[src[off[P]:off[P + 1]]], layer.epd_h[off[P]:off[P + 1]]) for P in range(E)]
    for e, rows, h in groups + [(E, x.astype(np.float64), layer.h_shared)]:
        h = h.float().cpu().numpy()
        g, u = rows @ wg[e].astype(np.float64).T, rows @ wu[e].astype(np.float64).T
        far = g < -100.0           # exp(-g) overflows f32 well before: the activation is 0
        assert far[:, :32].any() and np.array_equal(h[far], np.zeros(far.sum(), dtype=np.float32)), f"expert {e}"
        near = np.abs(u).max(axis=1) < 1e6
        g, u = g[near], u[near]
        assert_one_rounding(h[near], g / (1.0 + np.exp(-g)) * u, f"h of expert {e}")


def _rows_by_token_and_expert(layer):
    """EPD row of every (token, expert) pair of the layer's last plan."""
    tab = layer.tables()
    off, expert = tab["exp_offset"].cpu().numpy(), tab["pos_expert"].cpu().numpy()
    token = tab["sfd_token"].cpu().numpy()[tab["epd_sfd_row"].cpu().numpy()]
    return {(int(token[r]), int(expert[P])): r for P in range(len(expert)) for r in range(off[P], off[P + 1])}


def _bits(t):
    return t.view(torch.int16).cpu().numpy()


@pytest.mark.parametrize("T,part,d,f,E,S,k", [
    (160, 100, 512, 320, 8, 2, 1),    # 20 rows per expert, two K tiles per quarter
    (200, 100, 320, 448, 10, 2, 1),   # five K tiles: quarters of one and two
    (150, 100, 192, 192, 8, 3, 1),    # three K tiles: the quarters of K have none or one
    (300, 100, 512, 256, 40, 2, 3),
])
def test_few_rows_have_the_bits_of_smaller_batches(T, part, d, f, E, S, k):
    """The weight-streaming kernel, which takes the first `part` tokens alone, sums the gate/up product in quarters of K; the
    128-row tiles, which take all T beside their shared experts, sum the same quarters.  The stored activations and
    products of a token are the same bits, and a training step's are too."""
    say(f"rows of {part} and {T} tokens E={E} S={S} k={k} d={d} f={f}")
    dev = require_gpu()
    wk = wl.make_workload(wl.LayerShape("few", T=T, d=d, f=f, E=E, S=S, k=k, D=2, dtype="bf16", components=4), seed=T)
    lg, x = torch.from_numpy(wk.logits).to(dev), to_dev(wk.x, "bf16", dev)
    w = [to_dev(a, "bf16", dev) for a in (wk.w_gate, wk.w_up, wk.w_down)]
    small, whole = (OccultLayer(n, d, f, E, S, k, 2, "bf16") for n in (part, T))
    small.forward(lg[:part].contiguous(), x[:part].contiguous(), *w)
    for train in (False, True):
        whole.forward(lg, x, *w, train=train)
        torch.cuda.synchronize()
        at, ref = _rows_by_token_and_expert(whole), _rows_by_token_and_expert(small)
        rows = np.array([(at[key], r) for key, r in ref.items()])
        for name in ("epd_h", "epd_y"):
            got, want = _bits(getattr(whole, name))[rows[:, 0]], _bits(getattr(small, name))[rows[:, 1]]
            assert np.array_equal(got, want), (name, train, np.mean(got != want))


@pytest.mark.parametrize("T,d,f,E,S,k,D", [   # (one row tile per expert, on 256 CUs)
    (800, 192, 320, 128, 0, 4, 4),    # gate/up 384 tiles: a round and 128, cut in 256 halves, every sixth past the columns; three K tiles
    (800, 704, 192, 128, 0, 4, 4),    # down and dx 384; K of three tiles, and of two matrices
    (800, 704, 320, 120, 1, 4, 4),    # up to 381 with the shared expert's in front
    (800, 704, 192, 100, 3, 4, 4),    # down: 300 and 21 shared, whose K is three times as long and which stand for three tiles each; none in halves
    (800, 704, 192, 240, 3, 8, 4),    # down and dx: 720 and 21 that stand for three each; what is left of 783 in halves
    (800, 704, 192, 160, 2, 5, 4),    # down: 480 and 21 that stand for two each; what is left of 522 in halves
])
def test_last_tiles_in_halves(T, d, f, E, S, k, D):
    test_tile128_products(T, d, f, E, S, k, D)


def test_more_tiles_than_loads_usually_leave():
    """129 rows in each of sixteen groups: 288 gate/up tiles for 256 CUs where the launch expects 216, so without half tiles."""
    E = 16
    test_tile128_products(129 * E, 192, 1152, E, 0, 1, 4, np.eye(E, dtype=np.float32)[np.arange(129 * E) % E])


def test_last_tiles_in_halves_with_k_in_parts():
    test_few_rows_have_the_bits_of_smaller_batches(800, 100, 1024, 320, 118, 1, 3)   # 375 tiles, K in quarters


@pytest.mark.parametrize("T,d,f,E,S,k,apart", [
    (140, 512, 256, 16, 4, 4, True),     # four K tiles of its own against the sixteen of the shared down projection
    (160, 1024, 512, 60, 4, 4, True),    # below 24 rows per expert
    (150, 512, 256, 256, 4, 1, True),    # more experts than rows
    (1000, 256, 192, 4, 4, 1, False),
    (1000, 1024, 512, 60, 1, 6, False),
])
def test_long_shared_down_projection_is_split_in_scratch(T, d, f, E, S, k, apart):
    """A shared down projection whose K, as one block's chain of tiles, would outlast the launch is split over workgroups
    into the scratch; one that the routed experts' launch covers leaves the scratch alone."""
    say(f"scratch of the shared down projection T={T} d={d} f={f} E={E} S={S} k={k}")
    dev = require_gpu()
    wk = wl.make_workload(wl.LayerShape("scratch", T=T, d=d, f=f, E=E, S=S, k=k, D=2, dtype="bf16", components=4), seed=S)
    w = [to_dev(a, "bf16", dev) for a in (wk.w_gate, wk.w_up, wk.w_down)]
    layer = OccultLayer(T, d, f, E, S, k, 2, "bf16")
    layer.ffn_ws.fill_(float("nan"))
    layer.forward(torch.from_numpy(wk.logits).to(dev), to_dev(wk.x, "bf16", dev), *w)
    torch.cuda.synchronize()
    assert bool(torch.isnan(layer.ffn_ws).all()) != apart
    h, wd = layer.h_shared.double().cpu().numpy(), wk.w_down[E:].astype(np.float64)
    ref = sum(h[:, s * f:(s + 1) * f] @ wd[s].T for s in range(S))
    assert_one_rounding(layer.y_shared.double().cpu().numpy(), ref, "y shared")


def test_shared_down_projection_has_the_bits_of_the_split_product():
    """With scratch the shared down projection is summed in three parts of K: by the small tiles into the scratch where a
    single routed expert has all 1000 rows, in registers by the 128-row tiles where four share them."""
    T, d, f, S = 1000, 256, 192, 4
    say(f"shared down projection in parts T={T} d={d} f={f} S={S}")
    dev = require_gpu()
    wk = wl.make_workload(wl.LayerShape("parts", T=T, d=d, f=f, E=4, S=S, k=1, D=1, dtype="bf16", components=4), seed=8)
    x = to_dev(wk.x, "bf16", dev)
    w4 = [to_dev(a, "bf16", dev) for a in (wk.w_gate, wk.w_up, wk.w_down)]
    out = []
    for E, w in ((4, w4), (1, [t[3:].contiguous() for t in w4])):
        layer = OccultLayer(T, d, f, E, S, 1, 1, "bf16")
        assert layer.ffn_ws is not None
        layer.forward(torch.from_numpy(wk.logits[:, :E].copy()).to(dev), x, *w)
        torch.cuda.synchronize()
        out.append((_bits(layer.h_shared), _bits(layer.y_shared)))
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1]), np.mean(out[0][1] != out[1][1])


@pytest.mark.parametrize("train", [False, True])
def test_many_rows_have_the_bits_of_larger_batches(train):
    """Without shared experts the 128-row tiles take groups below 500 rows on average and the 256-row tiles the others: the
    stored activations, products and pre-activations of a token are the same bits on both sides of the line."""
    d, f, E, k, T = 256, 192, 8, 2, 2000
    say(f"rows of {T - 1} and {T} tokens E={E} k={k} train={train}")
    dev = require_gpu()
    wk = wl.make_workload(wl.LayerShape("many", T=T, d=d, f=f, E=E, S=0, k=k, D=2, dtype="bf16", components=4), seed=T)
    lg, x = torch.from_numpy(wk.logits).to(dev), to_dev(wk.x, "bf16", dev)
    w = [to_dev(a, "bf16", dev) for a in (wk.w_gate, wk.w_up, wk.w_down)]
    part, whole = (OccultLayer(n, d, f, E, 0, k, 2, "bf16") for n in (T - 1, T))
    part.forward(lg[:T - 1].contiguous(), x[:T - 1].contiguous(), *w, train=train)
    whole.forward(lg, x, *w, train=train)
    torch.cuda.synchronize()
    at, ref = _rows_by_token_and_expert(whole), _rows_by_token_and_expert(part)
    rows = np.array([(at[key], r) for key, r in ref.items()])
    for name in ("epd_h", "epd_y") + (("epd_gu",) if train else ()):
        got, want = _bits(getattr(whole, name))[rows[:, 0]], _bits(getattr(part, name))[rows[:, 1]]
        assert np.array_equal(got, want), (name, np.mean(got != want))


@pytest.mark.parametrize("T", [800, 1100])
def test_weights_read_once_give_the_same_bits(T):
    """Below 88 rows per expert, and with weights larger than the memory-side cache, the weights are requested as not to be
    kept: the rows of the first 500 tokens are those that the same tokens get in a batch of 800 or 1100."""
    d, f, E, k, part = 2048, 1408, 64, 6, 500
    say(f"weights read once: {part} and {T} tokens E={E} d={d} f={f}")
    dev = require_gpu()
    gen = torch.Generator(device=dev)
    gen.manual_seed(1)
    rand = lambda *shape: torch.randn(shape, device=dev, generator=gen)
    lg, x = rand(T, E), rand(T, d).bfloat16()
    w = [(rand(E, *s) / s[1] ** 0.5).bfloat16() for s in ((f, d), (f, d), (d, f))]
    small, whole = (OccultLayer(n, d, f, E, 0, k, 4, "bf16") for n in (part, T))
    small.forward(lg[:part].contiguous(), x[:part].contiguous(), *w)
    whole.forward(lg, x, *w)
    torch.cuda.synchronize()
    at, ref = _rows_by_token_and_expert(whole), _rows_by_token_and_expert(small)
    rows = np.array([(at[key], r) for key, r in ref.items()])
    for name in ("epd_h", "epd_y"):
        got, want = _bits(getattr(whole, name))[rows[:, 0]], _bits(getattr(small, name))[rows[:, 1]]
        assert np.array_equal(got, want), (name, np.mean(got != want))


def _even_logits(T, E, k, gen, dev):
    """Scores whose top k are k neighbouring experts, dealt out in turn: T * k / E rows in every group."""
    lg = torch.rand((T, E), device=dev, generator=gen)
    chosen = (torch.arange(T, device=dev)[:, None] * k + torch.arange(k, device=dev)[None]) % E
    return lg.scatter_add_(1, chosen, torch.full((T, k), 2.0, device=dev))


@pytest.mark.parametrize("E,S,D,train", [(64, 2, 4, False), (64, 2, 4, True), (70, 0, 2, False)])
def test_streamed_weights_with_last_tiles_in_halves(E, S, D, train):
    """500 tokens, 42 - 47 rows in every group, weights larger than the memory-side cache: both products stream them and have tiles in
    halves, beside shared experts with a tile of the down projection standing for two (in parts of K, with the layer's scratch).
    Every output is the f64 product of its stored operands rounded once."""
    T, d, f, k = 500, 2048, 1408, 6
    say(f"streamed weights and half tiles T={T} d={d} f={f} E={E} S={S} k={k} train={train}")
    dev = require_gpu()
    gen = torch.Generator(device=dev)
    gen.manual_seed(3)
    lg, x = _even_logits(T, E, k, gen, dev), torch.randn((T, d), device=dev, generator=gen).bfloat16()
    w = [torch.randn((E + S, *s), device=dev, generator=gen, dtype=torch.bfloat16).mul_(s[1] ** -0.5) for s in ((f, d), (f, d), (d, f))]
    layer = OccultLayer(T, d, f, E, S, k, D, "bf16")
    layer.forward(lg, x, *w, train=train)
    torch.cuda.synchronize()
    tab = layer.tables()
    off, expert, src = (tab[n].cpu().numpy() for n in ("exp_offset", "pos_expert", "epd_sfd_row"))
    assert set(np.diff(off)) <= {T * k // E, T * k // E + 1}
    f64 = lambda t: t.double().cpu().numpy()

    def check(tag, e, rows, h, gu):
        g, u = rows.double() @ w[0][e].double().T, rows.double() @ w[1][e].double().T
        assert_one_rounding(f64(h), f64(g / (1.0 + torch.exp(-g)) * u), f"h {tag}")
        if gu is not None:
            assert_one_rounding(f64(gu), f64(torch.cat([g, u], 1)), f"pre-activations {tag}")

    for P in range(E):
        r, e = slice(off[P], off[P + 1]), int(expert[P])
        check(f"expert {e}", e, layer.sfd_x[torch.from_numpy(src[r]).long().to(dev)], layer.epd_h[r], layer.epd_gu[r] if train else None)
        assert_one_rounding(f64(layer.epd_y[r]), f64(layer.epd_h[r].double() @ w[2][e].double().T), f"y expert {e}")
    y = 0
    for s in range(S):
        h = layer.h_shared[:, s * f:(s + 1) * f]
        check(f"shared {s}", E + s, x, h, layer.gu_shared[:, s * 2 * f:(s + 1) * 2 * f] if train else None)
        y = y + h.double() @ w[2][E + s].double().T
    if S:
        assert_one_rounding(f64(layer.y_shared), f64(y), "y shared")


def test_input_gradients_alone_are_those_of_a_training_step(monkeypatch):
    """130 rows per expert and weights larger than the memory-side cache: where weight gradients follow, the input gradients' products
    stream their weights, alone they do not; the last tiles in halves, a shared one standing for two.  Every output is the same bits,
    and the f64 product of its stored operands rounded once.  A layer expects weight gradients unless none followed the last time."""
    T, d, f, E, S, k = 520, 2048, 2688, 32, 2, 8
    say(f"input gradients alone T={T} d={d} f={f} E={E} S={S} k={k}")
    dev = require_gpu()
    gen = torch.Generator(device=dev)
    gen.manual_seed(2)
    rand = lambda *shape: torch.randn(shape, device=dev, generator=gen)
    lg, x, dy = _even_logits(T, E, k, gen, dev), rand(T, d).bfloat16(), rand(T, d).bfloat16()
    w = [torch.randn((E + S, *s), device=dev, generator=gen, dtype=torch.bfloat16).mul_(s[1] ** -0.5) for s in ((f, d), (f, d), (d, f))]
    layer = OccultLayer(T, d, f, E, S, k, 4, "bf16")
    layer.transpose_weights(*w)
    follow, call = [], B.occult_expert_ffn_backward
    monkeypatch.setattr(B, "occult_expert_ffn_backward", lambda *a, **kw: (follow.append(kw["weights_follow"]), call(*a, **kw)))
    names = ("epd_dh", "epd_gu", "epd_dx", "dh_shared", "gu_shared", "dx_shared")
    got = []
    for step in range(4):
        layer.forward(lg, x, *w, train=True)
        layer.backward_input(x, w[0], w[1], dy)
        if step < 2:
            torch.cuda.synchronize()
            got.append([getattr(layer, n).clone() for n in names])
        else:
            layer.expert_ffn_backward_weights(x, dy)
    torch.cuda.synchronize()
    assert follow == [True, False, False, True]
    for name, a, b in zip(names, *got):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), name
    off, expert = (layer.tables()[n].cpu().numpy() for n in ("exp_offset", "pos_expert"))
    assert set(np.diff(off)) == {T * k // E}
    dh, dgu, dx, dhs, dgus, dxs = got[0]
    f64 = lambda t: t.double().cpu().numpy()
    dx_ref = 0
    for P, e in [(P, int(expert[P])) for P in range(E)] + [(None, E + s) for s in range(S)]:
        wg, wu, wd = (t[e].double() for t in w)
        if P is not None:
            r = slice(off[P], off[P + 1])
            assert_one_rounding(f64(dh[r]), f64(layer.epd_dy[r].double() @ wd), f"dh expert {e}")
            assert_one_rounding(f64(dx[r]), f64(dgu[r, :f].double() @ wg + dgu[r, f:].double() @ wu), f"dx expert {e}")
        else:
            c = (e - E) * f
            assert_one_rounding(f64(dhs[:, c:c + f]), f64(dy.double() @ wd), f"dh shared {e}")
            dx_ref = dx_ref + dgus[:, 2 * c:2 * c + f].double() @ wg + dgus[:, 2 * c + f:2 * c + 2 * f].double() @ wu
    assert_one_rounding(f64(dxs), f64(dx_ref), "dx shared")
