"""The direct minibatch kernels (fragments straight from memory, chain step and gradients in one launch) at the edges of
their tiles and of the rules that choose them, against the oracle; and the same bits from every way to enqueue them."""
import numpy as np
import pytest

from lf_inputs import make_net, round_to_bf16
from tests.gpu_util import check_against_oracle, log, run_gpu, to_np

pytestmark = pytest.mark.gpu


def _tensors(g):
    return [to_np(t).view(np.uint32).copy() for t in g.nabla_w + g.nabla_b]


# of the nets below: those that lf_backward_leapfrog_noalloc is not published to serve
BEYOND_NOALLOC = [((3, 2056), 130), ((3, 4104), 64), ((3, 2056), 400), ((3, 3080), 200), ((64, 3076, 3076, 260), 64),
                  ((64, 4100, 4100, 200), 52)]


@pytest.mark.parametrize("shape,B,dtype", [
    ((3, 4), 2, "f32"),               # less than one tile and one unit of the contraction in every dimension
    ((3, 8), 1, "bf16"),
    ((5, 520), 37, "f32"),            # tiles of 16 x 16, a ragged third row block; gradients 32 x 32 a wave
    ((4, 520), 77, "f32"),            # gradients whose waves share the samples, a ragged last unit
    ((4, 520), 130, "bf16"),
    ((3, 2052), 15, "f32"),           # gradients 64 x 64 a wave, ragged edges of both kinds
    ((3, 2048), 64, "f32"),           # tiles of 16 x 32, all full
    ((4, 1032), 20, "bf16"),          # tiles of 16 x 16 and 16 x 32
    ((3, 1500), 100, "f32"),          # tiles of 32 x 32, a ragged fourth row block
    ((3, 2056), 130, "f32"),          # tiles of 32 x 64, rows of the last one past the minibatch
    ((3, 4104), 64, "bf16"),
    ((3, 2056), 400, "f32"),          # tiles of 64 x 64
    ((3, 3080), 200, "bf16"),
    ((72, 1000, 36, 1500, 8), 19, "f32"),      # contractions shorter than a turn of the waves; unequal widths
    ((264, 8, 2056, 136), 33, "bf16"),
    ((3, 2048), 128, "bf16"),         # tiles of 32 x 32, all full; gradients 64 x 64 a wave
    ((520, 1000, 1500, 1500, 700, 264), 100, "f32"),   # layers whose gradients are cut in different ways, the last two too
    ((520, 1000, 1504, 1504, 704, 264), 100, "bf16"),
    ((64, 3076, 3076, 260), 64, "f32"),        # descent step: gradients whose waves share the samples beside a split chain step,
    ((64, 4100, 4100, 200), 52, "f32"),        # of 32 x 64 and of 64 x 64 tiles
])
def test_direct_kernels_match_oracle_with_the_same_bits_from_every_schedule(monkeypatch, shape, B, dtype):
    import paper_1801_04928_amd as P
    import torch
    monkeypatch.setenv("LF_GEMM_BIG", "0")
    widths = shape if len(shape) > 2 else (shape[1],) * shape[0]
    L = len(widths)
    net = make_net(L, widths[0] if len(shape) == 2 else widths, B, dtype=dtype, seed=sum(widths) + B)
    g = run_gpu(net, 1)                                   # chain step and the gradients above it in one launch
    rep = check_against_oracle(net, g)
    log(f"direct kernels {shape} B={B} {dtype}: worst {rep['worst']:.2e}")
    want = _tensors(g)
    stream = torch.cuda.current_stream().cuda_stream
    ways = [(sched, k) for sched in (P.LF_SCHED_AUTO, P.LF_SCHED_STREAMS) for k in sorted({1, L - 1})]
    for sched, k in ways:                                 # STREAMS: every product a launch of its own
        g.set_schedule(sched)
        for t in g.nabla_w + g.nabla_b:
            t.fill_(float("nan"))
        g.forward()
        g.backward(k)
        torch.cuda.synchronize()
        assert all(np.array_equal(a, b) for a, b in zip(want, _tensors(g))), (sched, k)
    for t in g.nabla_w + g.nabla_b:
        t.fill_(float("nan"))
    g.forward()
    st = P.lf_backward_leapfrog_noalloc(g.handle, g.y.data_ptr(), 1, stream)
    assert st == (P.LF_EUNSUPPORTED if (shape, B) in BEYOND_NOALLOC else P.LF_OK), P.lf_last_error(g.handle)
    torch.cuda.synchronize()
    if st == P.LF_OK:
        assert all(np.array_equal(a, b) for a, b in zip(want, _tensors(g)))
    else:
        assert all(bool(torch.isnan(t).all()) for t in g.nabla_w + g.nabla_b)
    # the descent step: layer l's rides one launch later, layers 3 and 2 share the last one
    results = []
    for sched in (P.LF_SCHED_AUTO, P.LF_SCHED_STREAMS):
        g.load(net)
        if g.master_w is not None:
            for m, w in zip(g.master_w, g.w):
                m.copy_(w)
        g.set_schedule(sched)
        g.set_sgd(0.125)
        g.forward()
        g.backward(L - 1)
        torch.cuda.synchronize()
        results.append([to_np(t).copy() for t in g.w + g.b + (g.master_w or [])])
    # eta is a power of two: one rounding, of the exact difference; the bf16 weights are the masters' rounding
    old = [net.w(l) for l in range(2, L + 1)] + [net.b(l) for l in range(2, L + 1)]
    new = results[0] if dtype == "f32" else results[0][2 * L - 2:] + results[0][L - 1:2 * L - 2]
    for i, (o, n, grad) in enumerate(zip(old, new, want)):
        exact = o.astype(np.float64) - 0.125 * grad.view(np.float32).astype(np.float64)
        assert np.array_equal(n, exact.astype(np.float32).reshape(n.shape)), i
    if dtype == "bf16":
        for w, master in zip(results[0][:L - 1], new):
            assert np.array_equal(w, round_to_bf16(master))
    assert all(np.array_equal(a, b) for a, b in zip(*results))
    g.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tile_with_a_row_block_past_the_minibatch(dtype):
    """64 x 64 tiles for three row blocks of 16 samples (wider nets than 8192 take them)."""
    net = make_net(3, 8200, 41, dtype=dtype, seed=8241, cache=False)
    g = run_gpu(net, 1)
    rep = check_against_oracle(net, g, sample_tiles=(40, 64), rng=np.random.default_rng(5))
    log(f"N=8200 B=41 {dtype}: worst {rep['worst']:.2e}")
    g.close()


@pytest.mark.parametrize("shape,B,k", [
    ((3, 3072), 768, 2),                  # direct forward, wide-net backward, gradients streamed
    ((4, 256), 32768, 2),                 # wide-net forward, direct backward
    ((4, 4104), 304, 2),                  # wide-net backward with a workgroup per gradient tile (rows of no whole lines)
    ((2048, 4104, 2080, 2048), 1024, 2),  # streamed and per-tile gradients in one net
    ((3, 8120), 8, 2),                    # a handful of samples, rows of gradients that are no whole 64-byte pieces
])
def test_plans_that_mix_direct_and_wide_kernels_match_oracle(shape, B, k):
    import torch
    widths = shape if len(shape) > 2 else (shape[1],) * shape[0]
    net = make_net(len(widths), widths[0] if len(shape) == 2 else widths, B, dtype="bf16", seed=sum(widths) + B, cache=False)
    g = run_gpu(net, k)
    rep = check_against_oracle(net, g, sample_tiles=(24, 96), rng=np.random.default_rng(3))
    log(f"mixed plan {shape} B={B}: worst {rep['worst']:.2e}")
    want = _tensors(g)
    for t in g.nabla_w + g.nabla_b:
        t.fill_(float("nan"))
    g.forward()
    g.backward(1)
    torch.cuda.synchronize()
    assert all(np.array_equal(a, b) for a, b in zip(want, _tensors(g)))
    g.close()
