"""Chain products of few samples through wide layers, whose contraction is split over workgroups that meet in memory, at the
edges of the rule that splits them: against the oracle, and the same bits from every way to enqueue them."""
import numpy as np
import pytest

from lf_inputs import make_net
from tests.gpu_util import check_against_oracle, log, run_gpu, to_np

pytestmark = pytest.mark.gpu


def _tensors(g):
    return [to_np(t).view(np.uint32).copy() for t in g.nabla_w + g.nabla_b]


@pytest.mark.parametrize("widths,B,dtype", [
    ((1024,) * 4, 8, "bf16"),               # 16 x 32 tiles, four splits: the narrowest
    ((1288, 1032, 2048, 1024), 24, "bf16"),  # 32 x 32, four splits; ragged tiles and contractions; a whole step above it
    ((2184,) * 3, 16, "bf16"),              # 16 x 64, four splits
    ((2600,) * 3, 16, "bf16"),              # 16 x 64, two splits
    ((3080,) * 3, 19, "bf16"),              # 32 x 64, two splits
    ((3080,) * 3, 41, "bf16"),              # the same for three row blocks
    ((4096,) * 4, 64, "bf16"),              # 32 x 64, two splits, all of 256 workgroups
    ((4104,) * 3, 33, "bf16"),              # 64 x 64, two splits
    ((8192,) * 3, 40, "bf16"),              # 64 x 64, two splits, all of 256 workgroups, a row block past the minibatch
    ((1024, 1028, 1040, 1024), 2, "f32"),   # 16 x 32, four splits
    ((1024, 1028, 1500, 1024), 2, "f32"),   # whole steps: a turn more, a contraction shorter than the width
    ((2052,) * 3, 16, "f32"),               # 16 x 64, four splits
    ((3076,) * 3, 30, "f32"),               # 32 x 64, four splits
    ((3588,) * 3, 30, "f32"),               # 32 x 64, two splits
    ((4100, 3072, 4100), 37, "f32"),        # 32 x 64, two splits, a ragged second row block
    ((4100,) * 3, 64, "f32"),               # 64 x 64, two splits
    ((1020, 1024, 1024, 2048, 512), 16, "f32"),   # split and whole steps in one net
])
def test_split_chain_matches_oracle_with_the_same_bits_from_every_schedule(monkeypatch, widths, B, dtype):
    import paper_1801_04928_amd as P
    import torch
    monkeypatch.setenv("LF_GEMM_BIG", "0")
    L = len(widths)
    net = make_net(L, widths[0] if len(set(widths)) == 1 else widths, B, dtype=dtype, seed=sum(widths) + B, cache=False)
    g = run_gpu(net, 1)
    rep = check_against_oracle(net, g, sample_tiles=(24, 96), rng=np.random.default_rng(1))
    log(f"split chain {widths} B={B} {dtype}: worst {rep['worst']:.2e}")
    want = _tensors(g)

    def same(what):
        torch.cuda.synchronize()
        assert all(np.array_equal(a, b) for a, b in zip(want, _tensors(g))), what
        for t in g.nabla_w + g.nabla_b:
            t.fill_(float("nan"))

    def scribble():
        """Whatever the workspace holds when a forward and a backward pass begin, the arrival counters too."""
        torch.cuda.synchronize()
        g.workspace.fill_(255)

    for sched, k in ((P.LF_SCHED_AUTO, L - 1), (P.LF_SCHED_STREAMS, 1), (P.LF_SCHED_STREAMS, L - 1), (P.LF_SCHED_AUTO, 1)):
        g.set_schedule(sched)
        scribble()
        for _ in range(3):                                # pass after pass on the same counters
            g.forward()
            g.backward(k)
        same((sched, k))
    if min(widths) < 4096 or B <= 32:                     # (the others are beyond the published limit)
        scribble()
        for _ in range(2):
            g.forward()
            st = P.lf_backward_leapfrog_noalloc(g.handle, g.y.data_ptr(), 1, torch.cuda.current_stream().cuda_stream)
            assert st == P.LF_OK, P.lf_last_error(g.handle)
        same("noalloc")
    scribble()
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            g.forward()
            g.backward(1)
        for _ in range(3):
            graph.replay()
            same("replay")
            g.forward()
            g.backward(1)
            same("between replays")
    g.close()
