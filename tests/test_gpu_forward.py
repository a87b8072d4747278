"""layer.forward() is one call into the library: the same bits in every buffer as the five steps called one by one, for
each kind of expert computation, and the errors of the steps."""
import ctypes

import pytest
import torch

from inputs import workloads as wl
from paper_2505_13345_amd import binding as B
from paper_2505_13345_amd.layer import OccultLayer
from tests.helpers import require_gpu, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,S,dtype,n_d,packed,train", [
    (1, 2, "bf16", 0, True, False), (40, 0, "bf16", 2, True, False), (300, 2, "bf16", 0, False, False),
    (300, 2, "bf16", 0, True, True), (33, 0, "bf16", 0, False, True), (50, 1, "f32", 0, False, False),
    (50, 1, "f32", 0, False, True), (0, 1, "bf16", 0, False, False),
])
def test_forward_is_its_steps(T, S, dtype, n_d, packed, train):
    say(f"forward T={T} S={S} {dtype} n_d={n_d} packed={packed} train={train}")
    dev = require_gpu()
    d, f, E, k, D = 192, 128, 16, 4, 4
    wk = wl.make_workload(wl.LayerShape("fwd", T=max(T, 1), d=d, f=f, E=E, S=S, k=k, D=D, dtype=dtype, components=4), seed=T)
    x, lg = to_dev(wk.x, dtype, dev)[:T], torch.from_numpy(wk.logits).to(dev)[:T]
    w = [to_dev(a, dtype, dev) for a in (wk.w_gate, wk.w_up, wk.w_down)]
    one, steps = (OccultLayer(T, d, f, E, S, k, D, dtype, n_d=n_d) for _ in range(2))
    for layer in (one, steps):
        if packed:
            layer.pack_weights(*w)
    y = one.forward(lg, x, *w, train=train)
    steps.route(lg)
    steps.make_plan()
    steps.dispatch(x)
    (steps.expert_ffn_train if train else steps.expert_ffn)(x, *w)
    steps.combine()
    torch.cuda.synchronize()
    assert y is one.y and getattr(one, "gu_saved", False) == train
    for name in ("plan_mem", "ids", "w", "sfd_x", "sfd_y", "y", "epd_h", "epd_y", "h_shared", "y_shared", "epd_gu", "gu_shared"):
        a, b = getattr(one, name, None), getattr(steps, name, None)
        assert (a is None) == (b is None), name
        assert a is None or torch.equal(a.view(torch.uint8), b.view(torch.uint8)), name


def test_forward_refuses_what_its_steps_refuse():
    say("forward's errors")
    dev = require_gpu()
    layer = OccultLayer(8, 64, 64, 8, 0, 2, 2, "bf16")
    w = [torch.zeros((8, 64, 64), dtype=torch.bfloat16, device=dev) for _ in range(3)]
    lg, x = torch.zeros((8, 8), device=dev), torch.zeros((8, 64), dtype=torch.bfloat16, device=dev)
    for bad in ((lg[:4], x, *w), (lg, x.float(), *w), (lg, x, w[0][:7], w[1], w[2]), (lg, x, *w[:2], w[2].transpose(1, 2)),
                (lg.cpu(), x, *w)):
        with pytest.raises(ValueError):
            layer.forward(*bad)
    with pytest.raises(B.OccultError):   # no buffers for the experts
        OccultLayer(8, 64, 64, 8, 0, 2, 2, "bf16", with_ffn=False).forward(lg, x, *w)


@pytest.mark.parametrize("T,d,E,k,D,dtype", [
    (3, 64, 8, 2, 2, "f32"), (4, 512, 60, 4, 4, "bf16"), (5, 576, 64, 8, 64, "bf16"), (255, 2048, 64, 6, 16, "bf16"),
    (256, 2112, 16, 12, 1, "bf16"), (257, 4096, 20, 20, 5, "bf16"), (512, 1024, 256, 32, 64, "bf16"), (513, 64, 16, 4, 4, "bf16"),
    (7, 4160, 8, 2, 4, "bf16"),
])
def test_forward_of_small_batches(T, d, E, k, D, dtype):
    """Plan and row copies in one launch: tokens around a workgroup's four, a block of 256 and the last size, rows of one
    vector and fewer up to eight per lane and beyond, all devices, up to 32 slots; tables and rows as the separate calls'."""
    say(f"forward T={T} d={d} E={E} k={k} D={D} {dtype}")
    dev = require_gpu()
    gen = torch.Generator().manual_seed(T)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn((T, d), generator=gen).to(dt).to(dev)
    lg = torch.randn((T, E), generator=gen).to(dev)
    w = [torch.randn(s, generator=gen).mul_(0.05).to(dt).to(dev) for s in ((E, 64, d), (E, 64, d), (E, d, 64))]
    one, steps = (OccultLayer(T, d, 64, E, 0, k, D, dtype) for _ in range(2))
    one.forward(lg, x, *w)
    steps.route(lg)
    steps.make_plan()
    steps.dispatch(x)
    steps.expert_ffn(x, *w)
    steps.combine()
    torch.cuda.synchronize()
    for name in ("plan_mem", "ids", "w", "sfd_x", "y"):
        assert torch.equal(getattr(one, name).view(torch.uint8), getattr(steps, name).view(torch.uint8)), name


@pytest.mark.parametrize("T,d,f,E,S,k,D,n_d,mode,packed", [
    (1, 256, 64, 60, 4, 4, 4, 0, 1, True), (1, 64, 64, 2, 0, 1, 1, 0, 1, False), (2, 576, 128, 8, 1, 8, 2, 0, 1, False),
    (3, 4096, 64, 130, 0, 8, 10, 2, 1, False), (4, 192, 64, 256, 1, 8, 8, 2, 3, True), (4, 128, 64, 64, 0, 6, 16, 3, 2, False),
    (4, 2112, 192, 64, 2, 7, 64, 0, 1, True), (5, 704, 64, 64, 0, 8, 64, 0, 1, False), (8, 320, 192, 16, 2, 2, 4, 0, 1, True),
    (12, 1408, 384, 64, 1, 8, 8, 0, 1, False), (12, 128, 64, 61, 0, 3, 1, 0, 1, True),
    # routed and planned in launches of their own
    (13, 320, 64, 16, 2, 2, 4, 0, 1, True), (5, 128, 128, 65, 0, 3, 5, 0, 1, False), (5, 128, 128, 16, 0, 3, 4, 2, 1, False),
    (12, 256, 384, 64, 0, 8, 8, 0, 1, False), (4, 64, 64, 16, 0, 9, 4, 0, 1, False), (1, 4160, 64, 16, 1, 2, 4, 0, 1, True),
])
def test_forward_of_a_few_tokens(T, d, f, E, S, k, D, n_d, mode, packed):
    """Routing, plan, row copies and the gate/up product in one launch, and the sizes around it: every workgroup's own routing and row
    tiles (one or three rounds of tokens, pruned each way, ties, scores that are no numbers, experts placed anywhere, more than
    64 of them) give the bits of the separate steps in every buffer."""
    say(f"forward T={T} d={d} f={f} E={E} S={S} k={k} D={D} n_d={n_d} mode={mode} packed={packed}")
    dev = require_gpu()
    gen = torch.Generator().manual_seed(T * E + d)
    bf = lambda *shape: torch.randn(shape, generator=gen).mul_(0.1).to(torch.bfloat16).to(dev)
    x, w = bf(T, d), (bf(E + S, f, d), bf(E + S, f, d), bf(E + S, d, f))
    lg = torch.randn((T, E), generator=gen).mul_(2).round().mul_(0.5)   # many ties
    lg[0, 0], lg[T - 1, E - 1], lg[T // 2, E // 2] = float("nan"), float("inf"), float("-inf")
    lg = lg.to(dev)
    pos = torch.randperm(E, generator=gen).to(torch.int32)
    table = None
    if mode == 3:
        table = torch.stack([p[p != e] for e, p in ((e, torch.randperm(E, generator=gen)) for e in range(E))]).to(torch.int32)
    one, steps = (OccultLayer(T, d, f, E, S, k, D, "bf16", n_d, mode, 1, pos, sim_table=table) for _ in range(2))
    for layer in (one, steps):
        if packed:
            layer.pack_weights(*w)
    one.forward(lg, x, *w)
    steps.route(lg)
    steps.make_plan()
    steps.dispatch(x)
    steps.expert_ffn(x, *w)
    steps.combine()
    torch.cuda.synchronize()
    for name in ("plan_mem", "ids", "w", "sfd_x", "sfd_y", "y", "epd_h", "epd_y", "h_shared", "y_shared"):
        a, b = getattr(one, name), getattr(steps, name)
        assert a is None or torch.equal(a.view(torch.uint8), b.view(torch.uint8)), name


def _kernels_of(call):
    """Kernel launches of a call, counted as the nodes of its graph."""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    hip = ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))
    n = ctypes.c_size_t()
    assert hip.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("T,d,f,E,S,k,n_d,merged", [
    (1, 256, 64, 60, 4, 4, 0, True), (4, 192, 64, 256, 1, 8, 2, True), (12, 1408, 384, 64, 1, 8, 0, True),
    (13, 320, 64, 16, 2, 2, 0, False), (5, 128, 128, 65, 0, 3, 0, False), (5, 128, 128, 16, 0, 3, 2, False),
    (12, 256, 384, 64, 0, 8, 0, False), (4, 64, 64, 16, 0, 9, 0, False), (1, 4160, 64, 16, 1, 2, 0, False),
    # 2560 workgroups that route and one column block more; 6 d of them and more
    (4, 64, 2560, 32, 0, 8, 0, True), (4, 64, 2624, 32, 0, 8, 0, False),
    (4, 448, 2688, 32, 1, 8, 0, True), (4, 448, 2752, 32, 1, 8, 0, False),
])
def test_which_forward_passes_merge_their_first_launches(T, d, f, E, S, k, n_d, merged):
    say(f"launches of forward T={T} d={d} f={f} E={E} S={S} k={k} n_d={n_d}")
    dev = require_gpu()
    gen = torch.Generator(device=dev)
    gen.manual_seed(T + f)
    bf = lambda *shape: torch.randn(shape, device=dev, generator=gen).mul_(0.05).to(torch.bfloat16)
    x, w, lg = bf(T, d), (bf(E + S, f, d), bf(E + S, f, d), bf(E + S, d, f)), torch.randn((T, E), device=dev, generator=gen)
    one, steps = (OccultLayer(T, d, f, E, S, k, 4 if E % 4 == 0 else 5, "bf16", n_d) for _ in range(2))
    one.forward(lg, x, *w)
    steps.route(lg)
    steps.make_plan()
    steps.dispatch(x)
    steps.expert_ffn(x, *w)
    steps.combine()
    torch.cuda.synchronize()
    assert torch.equal(one.y.view(torch.int16), steps.y.view(torch.int16))
    launches = _kernels_of(lambda: one.forward(lg, x, *w))
    assert launches == 3 if merged else launches > 3


@pytest.mark.parametrize("S,one_call", [(0, True), (1, True), (0, False), (1, False)])
def test_kept_pre_activations_are_of_the_present_batch(S, one_call):
    """A training pass on one batch, a plain one on another, the backward on the latter: what a layer gives that has only
    seen the second batch (its pre-activations are recomputed), not the first batch's pre-activations in the second's rows."""
    say(f"pre-activations S={S} one_call={one_call}")
    dev = require_gpu()
    T, d, f, E, k, D = 96, 128, 64, 8, 2, 4
    gen = torch.Generator().manual_seed(S)
    bf = lambda *shape: torch.randn(shape, generator=gen).to(torch.bfloat16).to(dev)
    w = [bf(E + S, f, d) * 0.1, bf(E + S, f, d) * 0.1, bf(E + S, d, f) * 0.1]
    xa, xb, dy = bf(T, d), bf(T, d), bf(T, d)
    la, lb = (torch.randn((T, E), generator=gen).to(dev) for _ in range(2))
    both, fresh = (OccultLayer(T, d, f, E, S, k, D, "bf16") for _ in range(2))

    def plain(layer):
        if one_call:
            return layer.forward(lb, xb, *w)
        layer.route(lb)
        layer.make_plan()
        layer.dispatch(xb)
        layer.expert_ffn(xb, *w)
        layer.combine()

    both.forward(la, xa, *w, train=True)
    assert both.gu_saved
    got = []
    for layer in (both, fresh):
        plain(layer)
        layer.transpose_weights(*w)
        got.append(layer.backward_input(xb, w[0], w[1], dy) + layer.expert_ffn_backward_weights(xb, dy))
    torch.cuda.synchronize()
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("step", ["route", "make_plan", "dispatch", "expert_ffn", "expert_ffn_train", "combine"])
@pytest.mark.parametrize("where", ["subclass", "object", "class"])
def test_forward_goes_through_replaced_steps(step, where, monkeypatch):
    say(f"forward with its own {step} in the {where}")
    dev = require_gpu()
    T, d, f, E, k, D, train = 20, 64, 64, 8, 2, 4, step == "expert_ffn_train"
    gen = torch.Generator().manual_seed(1)
    bf = lambda *shape: torch.randn(shape, generator=gen).to(torch.bfloat16).to(dev)
    x, lg, w = bf(T, d), torch.randn((T, E), generator=gen).to(dev), (bf(E, f, d), bf(E, f, d), bf(E, d, f))
    want = OccultLayer(T, d, f, E, 0, k, D, "bf16").forward(lg, x, *w, train=train)
    own, calls = getattr(OccultLayer, step), []

    def replaced(self, *args):
        calls.append(step)
        return own(self, *args)

    layer = (type("Own", (OccultLayer,), {step: replaced}) if where == "subclass" else OccultLayer)(T, d, f, E, 0, k, D, "bf16")
    if where == "object":
        setattr(layer, step, replaced.__get__(layer))
    if where == "class":
        monkeypatch.setattr(OccultLayer, step, replaced)
    y = layer.forward(lg, x, *w, train=train)
    torch.cuda.synchronize()
    assert calls == [step] and layer.gu_saved == train
    assert torch.equal(y, want)
