"""Single-sample nets outside the persistent kernels' shapes, schedule left to the library: the gradients ride beside the chain
step of the layer below.  The same bits as the stream schedule's launches of their own, and the oracle's gradients."""
import numpy as np
import pytest

from lf_inputs import make_net
from tests.gpu_util import check_against_oracle, log, run_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths", [
    (4, 8),                                    # the persistent kernels' shape: no chain step
    (4100, 8), (8, 4100),                      # outside it, and no chain step
    (260, 4, 516),                             # one chain step, less than a row block
    (4100, 4100, 4100),                        # beyond the persistent kernels' width
    (8, 2052, 260, 4096, 12, 1000, 4, 256),    # chain steps of 4 and 16 rows a wave; strips and rows that end inside a block
    (8, 260, 2052, 1000, 12, 256),             # of 8 rows a wave, with the gradients or the descent step beside them
    (84, 996, 6348, 1364, 88),
])
def test_gradients_beside_the_chain_match_the_streams_and_the_oracle(widths):
    import paper_1801_04928_amd as P
    import torch
    L = len(widths)
    net = make_net(L, widths, 1, dtype="f32", seed=sum(widths), cache=False)
    g = run_gpu(net, L - 1)
    rep = check_against_oracle(net, g)
    log(f"single sample in line {widths}: worst {rep['worst']:.2e}")

    def run(sched, k, eta):
        g.load(net)
        g.set_schedule(sched)
        g.set_sgd(eta)
        for t in g.nabla_w + g.nabla_b:
            t.fill_(float("nan"))
        g.forward()
        g.backward(k)
        torch.cuda.synchronize()
        return [to_np(t).view(np.uint32).copy() for t in (g.w + g.b if eta else g.nabla_w + g.nabla_b)]

    for eta in (0.0, 0.125):
        want = run(P.LF_SCHED_STREAMS, 1, eta)
        for sched, k in ((P.LF_SCHED_AUTO, 1), (P.LF_SCHED_AUTO, L - 1), (P.LF_SCHED_STREAMS, L - 1)):
            assert all(np.array_equal(a, b) for a, b in zip(want, run(sched, k, eta))), (sched, k, eta)
    g.close()


@pytest.mark.parametrize("widths", [
    (2300, 8, 4092, 68, 1020, 4),      # a row a wave: what is left of a row 63, 2, 7 x 64 + 63, 17, 3 x 64 + 63 vectors of four
    (3000, 2504, 3008, 2560, 2048),    # two rows a wave: 3 x 64 + 46, 64 + 50, 3 x 64 - 16, 2 x 64
    (5000, 4100, 4612),                # a row a wave: 3 x 64 + 34, 1, after whole turns
])
def test_forward_rows_of_any_length_plain_and_non_temporal(monkeypatch, widths):
    """How a load is cached changes no value."""
    net = make_net(len(widths), widths, 1, dtype="f32", seed=sum(widths), cache=False)
    bits = []
    for stream in ("1", "0"):
        monkeypatch.setenv("LF_PERSISTENT_STREAM_WEIGHTS", stream)
        g = run_gpu(net, 1)
        rep = check_against_oracle(net, g)
        log(f"forward rows {widths}, streamed {stream}: worst {rep['worst']:.2e}")
        bits.append([to_np(g.activation(l)).view(np.uint32).copy() for l in range(2, len(widths) + 1)])
        g.close()
    assert all(np.array_equal(a, b) for a, b in zip(*bits))
