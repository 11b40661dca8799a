"""The backward entry point that allocates nothing (lf_backward_leapfrog_noalloc), called through the C ABI:
its gradients against lf_backward_leapfrog's on the same handle, bit for bit (the same kernels in the same
order) and hence within the parity tolerance, on two calls in a row, the second on a smaller net; then
minibatch nets, a shape beyond the published limit, and the oracle."""
import numpy as np
import pytest

from lf_inputs import make_net
from tests.gpu_util import TOL, check_against_oracle, poison_buffers, to_np

pytestmark = pytest.mark.gpu


def _run_pair(L, N, B, dtype, k, seed):
    """Gradients of lf_backward_leapfrog (stream schedule) and of the no-alloc call, same handle, same inputs."""
    import torch
    import paper_1801_04928_amd as P
    net = make_net(L, N, B, dtype=dtype, seed=seed)
    g = P.LeapfrogNet(L, N, B, dtype)
    g.load(net)
    g.set_schedule(P.LF_SCHED_STREAMS)
    stream = torch.cuda.current_stream().cuda_stream
    poison_buffers(g)
    assert P.lf_forward(g.handle, g.x.data_ptr(), stream) == P.LF_OK, P.lf_last_error(g.handle)
    assert P.lf_backward_leapfrog(g.handle, g.y.data_ptr(), k, stream) == P.LF_OK, P.lf_last_error(g.handle)
    torch.cuda.synchronize()
    want = [to_np(t).copy() for t in g.nabla_w + g.nabla_b]
    poison_buffers(g, whole_workspace=False)
    assert P.lf_forward(g.handle, g.x.data_ptr(), stream) == P.LF_OK
    st = P.lf_backward_leapfrog_noalloc(g.handle, g.y.data_ptr(), k, stream)
    assert st == P.LF_OK, P.lf_last_error(g.handle)
    torch.cuda.synchronize()
    got = [to_np(t).copy() for t in g.nabla_w + g.nabla_b]
    return net, g, want, got


def _assert_same(want, got, tol):
    for i, (a, b) in enumerate(zip(want, got)):
        assert np.all(np.isfinite(b)), f"tensor {i}: non-finite"
        scale = float(np.max(np.abs(a)))
        assert float(np.max(np.abs(a.astype(np.float64) - b))) <= tol * scale, f"tensor {i}: beyond the tolerance"
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32)), f"tensor {i}: bits differ"


def test_noalloc_backward_twice_second_call_smaller():
    import paper_1801_04928_amd as P
    assert P.lf_noalloc_scratch_limit() == 8 << 20
    net1, g1, want1, got1 = _run_pair(6, 2052, 1, "f32", 3, seed=11)      # 33 row blocks of partial sums
    _assert_same(want1, got1, TOL["f32"])
    net2, g2, want2, got2 = _run_pair(5, 516, 1, "f32", 2, seed=12)       # smaller: reuses the head of the scratch
    _assert_same(want2, got2, TOL["f32"])
    check_against_oracle(net2, g2)
    # the first handle again, after the smaller call has overwritten part of the scratch
    import torch
    stream = torch.cuda.current_stream().cuda_stream
    poison_buffers(g1, whole_workspace=False)
    assert P.lf_forward(g1.handle, g1.x.data_ptr(), stream) == P.LF_OK
    assert P.lf_backward_leapfrog_noalloc(g1.handle, g1.y.data_ptr(), 1, stream) == P.LF_OK
    torch.cuda.synchronize()
    _assert_same(want1, [to_np(t) for t in g1.nabla_w + g1.nabla_b], TOL["f32"])
    check_against_oracle(net1, g1)
    g1.close()
    g2.close()


@pytest.mark.parametrize("L,N,B,dtype,k", [(5, 512, 256, "f32", 4), (4, 264, 70, "bf16", 2),
                                           (3, 1856, 4096, "bf16", 2)])      # (wide-net kernels, no product split)
def test_noalloc_backward_minibatch(L, N, B, dtype, k):
    net, g, want, got = _run_pair(L, N, B, dtype, k, seed=N + B)
    _assert_same(want, got, TOL[dtype])
    check_against_oracle(net, g)
    g.close()


def test_noalloc_backward_limits():
    import torch
    import paper_1801_04928_amd as P
    stream = torch.cuda.current_stream().cuda_stream
    # a shape charged for more (8 x 256 x 4096 floats of split-K partials) than the static 8 MiB
    net = make_net(3, 4096, 256, seed=1, cache=False)
    g = P.LeapfrogNet(3, 4096, 256, "f32")
    g.load(net)
    assert P.lf_backward_leapfrog_noalloc(g.handle, g.y.data_ptr(), 1, stream) == P.LF_ESTATE      # no forward yet
    g.forward()
    assert P.lf_backward_leapfrog_noalloc(g.handle, g.y.data_ptr(), 1, stream) == P.LF_EUNSUPPORTED
    assert "static scratch" in P.lf_last_error(g.handle)
    assert P.lf_backward_leapfrog_noalloc(g.handle, g.y.data_ptr(), 3, stream) == P.LF_EINVAL     # k > L-1
    g.backward(1)                                    # the ordinary call still serves the shape
    torch.cuda.synchronize()
    g.close()
    assert P.lf_backward_leapfrog_noalloc(None, 0, 1, 0) == P.LF_EINVAL
