"""The small minibatch nets' kernels (one launch walks all layers, samples in slices) at the edges of their tiles, units,
slices and launches, against the oracle; the same bits from every schedule, from workgroups that draw their tasks, and from
replays of a captured pass."""
import numpy as np
import pytest

from lf_inputs import make_net
from tests.gpu_util import check_against_oracle, log, run_gpu, to_np

pytestmark = pytest.mark.gpu


def _bits(g):
    g.torch.cuda.synchronize()
    return [to_np(t).view(np.uint32).copy() for t in g.nabla_w + g.nabla_b]


def _again(g, k=1):
    for t in g.nabla_w + g.nabla_b:
        t.fill_(float("nan"))
    g.forward()
    g.backward(k)
    return _bits(g)


@pytest.mark.parametrize("shape,B,dtype", [
    ((5, 4), 2, "f32"),                # a tile and a unit that are mostly padding, a sample a slice
    ((5, 8), 1, "bf16"),
    ((6, 16), 8, "f32"),               # exactly a tile, eight slices of one sample
    ((6, 32), 9, "bf16"),
    ((5, 20), 17, "f32"),              # a tile and a quarter; slices of three samples, the last cluster empty
    ((5, 40), 19, "bf16"),
    ((5, 64), 128, "f32"),             # a unit a wave, full slices
    ((5, 132), 129, "f32"),            # three units for some waves; two slices a cluster
    ((5, 264), 131, "bf16"),
    ((5, 192), 40, "f32"),             # every instance of the contraction's length
    ((5, 256), 33, "f32"),
    ((5, 388), 12, "f32"),
    ((5, 512), 130, "f32"),            # the widest, two tasks a workgroup
    ((5, 384), 16, "bf16"),
    ((5, 776), 7, "bf16"),
    ((5, 1024), 144, "bf16"),
    ((5, 256), 520, "f32"),            # five slices a cluster
    ((8, 36, 500, 4, 260, 132, 512, 20), 21, "f32"),       # unequal widths, up and down
    ((8, 40, 1000, 8, 264, 136, 1024, 24), 37, "bf16"),
    ((67, 24), 5, "f32"),              # more steps than a launch holds
])
def test_small_nets_match_oracle_with_the_same_bits_from_every_schedule(monkeypatch, shape, B, dtype):
    import paper_1801_04928_amd as P
    monkeypatch.setenv("LF_CLUSTER", "1")
    widths = shape if len(shape) > 2 else (shape[1],) * shape[0]
    L = len(widths)
    net = make_net(L, widths[0] if len(shape) == 2 else widths, B, dtype=dtype, seed=sum(widths) + B)
    g = run_gpu(net, 1)
    rep = check_against_oracle(net, g)
    log(f"small nets {shape} B={B} {dtype}: worst {rep['worst']:.2e}")
    want = _bits(g)
    for sched in (P.LF_SCHED_AUTO, P.LF_SCHED_STREAMS):
        g.set_schedule(sched)
        for k in sorted({1, 3, L - 1}):
            assert all(np.array_equal(a, b) for a, b in zip(want, _again(g, k))), (sched, k)
    for t in g.nabla_w + g.nabla_b:
        t.fill_(float("nan"))
    g.forward()
    st = P.lf_backward_leapfrog_noalloc(g.handle, g.y.data_ptr(), 1, g.torch.cuda.current_stream().cuda_stream)
    assert st == P.LF_OK, P.lf_last_error(g.handle)
    assert all(np.array_equal(a, b) for a, b in zip(want, _bits(g)))
    g.close()
    # no cluster is ever complete: its workgroups draw their tasks in order
    monkeypatch.setenv("LF_CLUSTER_INCOMPLETE", "1")
    g = run_gpu(net, 1)
    for _ in range(2):
        assert all(np.array_equal(a, b) for a, b in zip(want, _again(g)))
    g.close()


def test_more_bf16_layers_than_a_launch_holds(monkeypatch):
    """Against a launch a layer: bfloat16 rounds a^l and delta^l to 2^-9 in each of 2 (L - 1) steps, and independent roundings add
    up as their root, 2.2e-2 at L = 67; two passes that round differently may be twice as far from each other."""
    import paper_1801_04928_amd as P
    net = make_net(67, 24, 5, dtype="bf16", seed=12)
    got = []
    for choice in ("0", "1"):
        monkeypatch.setenv("LF_CLUSTER", choice)
        g = P.LeapfrogNet(67, 24, 5, "bf16")
        g.load(net)
        g.set_cost_scale(66)                  # (delta shrinks by about four from layer to layer)
        g.forward()
        g.backward(1)
        g.torch.cuda.synchronize()
        got.append([to_np(t).astype(np.float64) for t in g.nabla_w + g.nabla_b])
        g.close()
    for want, have in zip(*got):
        assert np.abs(have - want).max() <= 2 * 2.0 ** -9 * (2 * 66) ** 0.5 * np.abs(want).max()


@pytest.mark.parametrize("widths,B,dtype", [((256,) * 8, 32, "f32"), ((512,) * 6, 100, "bf16"), ((36, 260, 100, 512, 64, 20), 21, "f32")])
def test_descent_step_of_a_small_net(monkeypatch, widths, B, dtype):
    """w - eta nabla_w with one rounding of the exact difference (eta is a power of two), from the gradients of the same pass."""
    import paper_1801_04928_amd as P
    monkeypatch.setenv("LF_CLUSTER", "1")
    L = len(widths)
    net = make_net(L, widths, B, dtype=dtype, seed=3)
    g = run_gpu(net, 1)
    grads = [to_np(t).copy() for t in g.nabla_w + g.nabla_b]
    old = [net.w(l) for l in range(2, L + 1)] + [net.b(l) for l in range(2, L + 1)]
    for sched in (P.LF_SCHED_AUTO, P.LF_SCHED_STREAMS):
        g.load(net)
        g.set_schedule(sched)
        g.set_sgd(0.125)
        g.forward()
        g.backward(2)
        g.torch.cuda.synchronize()
        for o, t, d in zip(old, (g.master_w or g.w) + g.b, grads):
            exact = o.astype(np.float64) - 0.125 * d.astype(np.float64)
            assert np.array_equal(to_np(t), exact.astype(np.float32).reshape(o.shape))
    g.close()


def test_bf16_weights_follow_their_masters(monkeypatch):
    """The weights that the next pass multiplies with are the stepped masters, rounded to nearest even: three steps in a row, each from
    the gradients of a net that starts with the same weights."""
    import paper_1801_04928_amd as P
    import torch
    monkeypatch.setenv("LF_CLUSTER", "1")
    L, N, B = 6, 520, 100
    net = make_net(L, N, B, dtype="bf16", seed=4)
    g, fresh = P.LeapfrogNet(L, N, B, "bf16"), P.LeapfrogNet(L, N, B, "bf16")
    for h in (g, fresh):
        h.load(net)
        h.set_sgd(0.125)
    tensors = lambda h: h.w + h.master_w + h.b  # noqa: E731
    for _ in range(3):
        before = [t.clone() for t in tensors(g)]
        for a, b in zip(tensors(fresh), before):
            a.copy_(b)
        fresh.set_sgd(0.0)
        fresh.forward()
        fresh.backward(1)
        g.forward()
        g.backward(1)
        torch.cuda.synchronize()
        for w, m, old, d in zip(g.w, g.master_w, before[L - 1:], fresh.nabla_w):
            exact = old.double() - 0.125 * d.double()          # (eta is a power of two: one rounding)
            assert torch.equal(m, exact.float()) and torch.equal(w, m.to(torch.bfloat16)) and not torch.equal(m, old)
    fresh.close()
    g.close()


def test_passes_of_several_nets_overlap(monkeypatch):
    """Nets that fill the compute units, each on a stream of its own, pass after pass without a wait between: their workgroups are not
    all resident at once, and nothing of one shows in another."""
    import torch
    monkeypatch.setenv("LF_CLUSTER", "1")
    shapes = [(8, 512, 128, "f32"), (8, 1024, 128, "bf16"), (8, 512, 300, "f32"), (12, 256, 512, "f32")]
    nets = [make_net(L, N, B, dtype=dtype, seed=L + B) for L, N, B, dtype in shapes]
    handles = [run_gpu(net, 1) for net in nets]
    want = [_bits(g) for g in handles]
    streams = [torch.cuda.Stream() for _ in handles]
    for g in handles:
        for t in g.nabla_w + g.nabla_b:
            t.fill_(float("nan"))
    torch.cuda.synchronize()
    for _ in range(20):
        for g, stream in zip(handles, streams):
            with torch.cuda.stream(stream):
                g.forward()
                g.backward(1)
    torch.cuda.synchronize()
    for g, w in zip(handles, want):
        assert all(np.array_equal(a, b) for a, b in zip(w, _bits(g)))
        g.grads(2)                     # (raises where a wait has given up)
        g.close()


def test_replays_of_a_captured_pass_beside_eager_ones(monkeypatch):
    """Captured before the handle's first pass and after it; replays with eager passes of the same handle in between."""
    import paper_1801_04928_amd as P
    import torch
    monkeypatch.setenv("LF_CLUSTER", "1")
    net = make_net(6, 200, 21, dtype="f32", seed=8)
    g = run_gpu(net, 1)
    want = _bits(g)
    g.close()
    g = P.LeapfrogNet(6, 200, 21, "f32")
    g.load(net)
    graphs = []
    for _ in range(2):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            g.forward()
            g.backward(1)
        graphs.append(graph)
        for _ in range(3):
            for graph in graphs:
                for t in g.nabla_w + g.nabla_b:
                    t.fill_(float("nan"))
                graph.replay()
                assert all(np.array_equal(a, b) for a, b in zip(want, _bits(g)))
            assert all(np.array_equal(a, b) for a, b in zip(want, _again(g, 2)))
    g.close()


def test_infinities_and_nans_stay_in_their_sample(monkeypatch):
    """A sample whose input is NaN or infinite leaves the other samples' activations and errors alone."""
    monkeypatch.setenv("LF_CLUSTER", "1")
    net = make_net(6, 132, 19, dtype="f32", seed=5)
    g = run_gpu(net, 1)
    a = [to_np(g.activation(l)).copy() for l in range(2, 7)]
    d = [to_np(g.delta(l)).copy() for l in range(2, 7)]
    g.x[4, 7] = float("nan")
    g.x[11, 0] = float("inf")
    g.forward()
    g.backward(1)
    g.torch.cuda.synchronize()
    others = [b for b in range(19) if b not in (4, 11)]
    for l in range(2, 7):
        assert np.array_equal(to_np(g.activation(l))[others], a[l - 2][others])
        assert np.array_equal(to_np(g.delta(l))[others], d[l - 2][others])
    assert np.isnan(to_np(g.activation(6))[4]).all() and np.isnan(to_np(g.delta(2))[4]).all()
    g.close()


def _on_workspace(g, workspace):
    """The same net on a handle that works in this workspace."""
    import paper_1801_04928_amd as P
    P.lf_destroy(g.handle)
    g.workspace = workspace
    st, g.handle = P.lf_create(g.L, g.N, g.B, g.dt, P.LF_COST_QUADRATIC, workspace.data_ptr(), workspace.numel())
    assert st == P.LF_OK, P.lf_last_error(None)
    pointers = lambda tensors: [t.data_ptr() for t in tensors]  # noqa: E731
    assert P.lf_set_params(g.handle, pointers(g.w), pointers(g.b)) == P.LF_OK
    assert P.lf_set_grad_buffers(g.handle, pointers(g.nabla_w), pointers(g.nabla_b)) == P.LF_OK


def test_the_workspace_may_hold_anything_when_a_pass_begins(monkeypatch):
    """Other values between the passes (words that carry tags of a pass too), eager and in a graph captured as the handle's
    first pass; and handles of other shapes and types that take turns on one workspace."""
    import paper_1801_04928_amd as P
    import torch
    monkeypatch.setenv("LF_CLUSTER", "1")
    shapes = [(6, 200, 21, "f32"), (5, 256, 40, "bf16"), (9, 64, 130, "f32")]
    nets = [make_net(L, N, B, dtype=dtype, seed=L) for L, N, B, dtype in shapes]
    handles = [run_gpu(net, 1) for net in nets]
    want = [_bits(g) for g in handles]
    workspace = torch.empty(max(g.workspace.numel() for g in handles), dtype=torch.uint8, device="cuda")
    for g in handles:
        _on_workspace(g, workspace)
    for _ in range(3):
        for g, w in zip(handles, want):
            assert all(np.array_equal(a, b) for a, b in zip(w, _again(g, 2)))
    g, w = handles[0], want[0]
    words = workspace[: workspace.numel() // 8 * 8].view(torch.int64)
    for value in (-1, 0, 1, *(tag << 32 for tag in range(1, 16)), 0x0000000200000002):
        words.fill_(value)
        assert all(np.array_equal(a, b) for a, b in zip(w, _again(g))), hex(value)
    _on_workspace(g, workspace)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.forward()
        g.backward(1)
    for value in (-1, 0x0000000200000002, 3 << 32, 0):
        words.fill_(value)
        for t in g.nabla_w + g.nabla_b:
            t.fill_(float("nan"))
        graph.replay()
        assert all(np.array_equal(a, b) for a, b in zip(w, _bits(g))), hex(value)
    for g in handles:
        g.close()


@pytest.mark.parametrize("sched", ["AUTO", "STREAMS"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_a_wait_that_gives_up_is_reported_and_takes_no_step(monkeypatch, dtype, sched):
    """No poll is repeated, and workgroups that draw their tasks are ahead of others' results: some wait gives up at once (the kernels
    end normally).  The descent step leaves the weights alone, the next call says so, and the handle's later passes are right."""
    import paper_1801_04928_amd as P
    import torch
    monkeypatch.setenv("LF_CLUSTER", "1")
    monkeypatch.setenv("LF_CLUSTER_SPIN_LIMIT", "0")
    monkeypatch.setenv("LF_CLUSTER_INCOMPLETE", "1")
    net = make_net(8, 256, 128, dtype=dtype, seed=6)
    g = P.LeapfrogNet(8, 256, 128, dtype)
    g.load(net)
    g.set_schedule(getattr(P, "LF_SCHED_" + sched))
    g.set_sgd(0.125)
    before = [t.clone() for t in g.w + g.b + (g.master_w or [])]
    g.forward()
    g.backward(2)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(before, g.w + g.b + (g.master_w or [])))
    with pytest.raises(P.LfError) as e:
        g.forward()
    assert e.value.status == P.LF_EHIP and "gave up" in str(e.value)
    with pytest.raises(P.LfError) as e:
        g.backward(1)
    assert e.value.status == P.LF_ESTATE
    g.set_sgd(0.0)
    g.forward()
    g.backward(2)
    torch.cuda.synchronize()
    check_against_oracle(net, g)
    g.close()


@pytest.mark.parametrize("widths,B,dtype", [
    ((256,) * 8, 32, "f32"), ((64, 64, 64, 64, 512, 64, 64, 64), 32, "f32"), ((784,) + (256,) * 6 + (16,), 32, "bf16")])
def test_small_nets_as_they_are_chosen(widths, B, dtype):
    """No choice forced: nets whose two directions, and nets whose chain alone, take these kernels, from any workspace, eager and replayed."""
    import torch
    net = make_net(len(widths), widths, B, dtype=dtype, seed=B)
    g = run_gpu(net, 1)
    check_against_oracle(net, g)
    want = _bits(g)
    for k in (1, 3):
        g.workspace.fill_(255)
        assert all(np.array_equal(a, b) for a, b in zip(want, _again(g, k))), k
    for _ in range(2):                 # backward passes of one forward pass
        g.backward(1)
        assert all(np.array_equal(a, b) for a, b in zip(want, _bits(g)))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.forward()
        g.backward(1)
    for _ in range(3):
        g.workspace.fill_(255)
        for t in g.nabla_w + g.nabla_b:
            t.fill_(float("nan"))
        graph.replay()
        assert all(np.array_equal(a, b) for a, b in zip(want, _bits(g)))
        assert all(np.array_equal(a, b) for a, b in zip(want, _again(g)))
    g.close()
