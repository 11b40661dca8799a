"""Several nets on one device: passes from several caller streams and threads, with one net captured or destroyed
meanwhile, give the bits of each net's sequential pass."""
import threading

import numpy as np
import pytest

from lf_inputs import make_net
from tests.gpu_util import run_gpu, to_np

pytestmark = pytest.mark.gpu


class _Thread(threading.Thread):
    """A thread whose exception is raised where it is joined."""

    def run(self):
        self.error = None
        try:
            super().run()
        except BaseException as e:  # noqa: BLE001
            self.error = e

    def join(self, timeout=None):
        super().join(timeout)
        if self.error is not None:
            raise self.error


def _bits(g):
    return [to_np(t).view(np.uint32).copy() for t in g.nabla_w + g.nabla_b]


def _clear(g):
    for t in g.nabla_w + g.nabla_b:
        t.fill_(float("nan"))


def _same(g, want):
    return all(np.array_equal(a, b) for a, b in zip(want, _bits(g)))


def test_nets_used_together_keep_their_bits():
    import paper_1801_04928_amd as P
    import torch
    shapes = [(6, 516, 1, "f32", 5), (5, 264, 37, "f32", 3), (4, 520, 40, "bf16", 2), (7, 260, 1, "f32", 2)]
    nets, want = [], []
    for L, N, B, dtype, k in shapes:
        g = run_gpu(make_net(L, N, B, dtype=dtype, seed=N + L), 1)
        g.set_schedule(P.LF_SCHED_STREAMS)          # (a single sample's sums have another order in the persistent kernels)
        g.forward()
        g.backward(1)
        torch.cuda.synchronize()
        want.append(_bits(g))
        nets.append(g)
    streams = [torch.cuda.Stream() for _ in nets]

    def passes(i, n):
        with torch.cuda.stream(streams[i]):
            for _ in range(n):
                nets[i].forward()
                nets[i].backward(shapes[i][4])

    for g in nets:
        _clear(g)
    torch.cuda.synchronize()
    threads = [_Thread(target=passes, args=(i, 5)) for i in range(len(nets))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert all(_same(g, w) for g, w in zip(nets, want))
    # another net's eager pass may be enqueued while a pass is being captured
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=streams[0], capture_error_mode="thread_local"):
        nets[0].forward()
        nets[0].backward(5)
        other = _Thread(target=passes, args=(1, 1))
        other.start()
        other.join()
    torch.cuda.synchronize()
    for replay in range(3):
        _clear(nets[0])
        _clear(nets[1])
        torch.cuda.synchronize()
        graph.replay()
        passes(1, 1)
        torch.cuda.synchronize()
        assert _same(nets[0], want[0]) and _same(nets[1], want[1]), replay
    # a destroyed net takes nothing from the others
    nets[0].close()
    for i in (1, 2, 3):
        _clear(nets[i])
        torch.cuda.synchronize()
        passes(i, 2)
        torch.cuda.synchronize()
        assert _same(nets[i], want[i]), i
        nets[i].close()
    g = run_gpu(make_net(6, 516, 1, seed=522), 1)               # nor the last one from the next
    g.set_schedule(P.LF_SCHED_STREAMS)
    _clear(g)
    g.forward()
    g.backward(5)
    torch.cuda.synchronize()
    assert _same(g, want[0])
    g.close()


def test_nets_on_one_stream_keep_their_bits():
    """Nets driven from one stream share worker streams: from several threads, with one of them on another stream too,
    captured there, or destroyed meanwhile."""
    import paper_1801_04928_amd as P
    import torch
    shapes = [(6, 516, 1, "f32", 5), (5, 264, 37, "f32", 3), (4, 520, 40, "bf16", 2), (7, 260, 1, "f32", 6)]
    home, away = torch.cuda.Stream(), torch.cuda.Stream()
    nets, want = [], []
    for L, N, B, dtype, k in shapes:
        g = run_gpu(make_net(L, N, B, dtype=dtype, seed=N + L), 1)
        g.set_schedule(P.LF_SCHED_STREAMS)
        g.forward()
        g.backward(1)
        torch.cuda.synchronize()
        want.append(_bits(g))
        nets.append(g)

    def passes(i, n, stream):
        with torch.cuda.stream(stream):
            for _ in range(n):
                nets[i].forward()
                nets[i].backward(shapes[i][4])

    def together(which, n):
        for i in which:
            _clear(nets[i])
        torch.cuda.synchronize()
        threads = [_Thread(target=passes, args=(i, n, home)) for i in which]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
        assert all(_same(nets[i], want[i]) for i in which)

    together(range(4), 1)
    together(range(4), 5)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=away, capture_error_mode="thread_local"):
        nets[0].forward()
        nets[0].backward(5)
        other = _Thread(target=passes, args=(1, 1, home))
        other.start()
        other.join()
    for replay in range(3):
        _clear(nets[0])
        torch.cuda.synchronize()
        with torch.cuda.stream(away):
            graph.replay()
        together((1, 2, 3), 2)
        assert _same(nets[0], want[0]), replay
    _clear(nets[0])
    torch.cuda.synchronize()
    passes(0, 2, away)
    together((1, 2), 2)
    assert _same(nets[0], want[0])
    nets[0].close()
    together((1, 2, 3), 2)
    for g in nets[1:]:
        g.close()
