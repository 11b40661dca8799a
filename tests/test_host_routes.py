"""Which kernels a net's passes launch, and which nets lf_backward_leapfrog_noalloc serves, from the calls the library makes
on the host (no kernel runs)."""
import re

import pytest

from tests import host_hip

# argv: widths, B, dtype, k, and "sgd" for the descent step.  Prints the kernels of a forward pass, of a backward pass, the status of the
# no-alloc backward pass, and the kernels of one more forward pass.
MAIN = r"""
#include <sstream>
int main(int argc, char** argv) {
    std::vector<int> n;
    std::stringstream widths(argv[1]);
    for (std::string w; std::getline(widths, w, '-');) n.push_back(std::atoi(w.c_str()));
    lf_net* net = make(n, std::atoi(argv[2]), argv[3][0] == 'b' ? LF_BF16 : LF_F32, LF_SCHED_AUTO);
    if (argc > 5) {                                       // the descent step
        std::vector<float*> masters(n.size(), (float*)some_input);
        if (argv[3][0] == 'b') CHECK(lf_set_master_weights(net, masters.data()) == LF_OK);
        CHECK(lf_set_sgd(net, 0.125f) == LF_OK);
    }
    auto print = [&](const char* what) {
        for (const std::string& s : launched) std::printf("%s %s\n", what, s.c_str());
        launched.clear();
    };
    CHECK(lf_forward(net, some_input, &caller_1) == LF_OK);
    print("forward");
    CHECK(lf_backward_leapfrog(net, some_input, std::atoi(argv[4]), &caller_1) == LF_OK);
    print("backward");
    std::printf("noalloc %d\n", (int)lf_backward_leapfrog_noalloc(net, some_input, 1, &caller_1));
    launched.clear();
    CHECK(lf_forward(net, some_input, &caller_1) == LF_OK);
    print("again");
    lf_destroy(net);
    return failures != 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return host_hip.build(tmp_path_factory.mktemp("routes"), MAIN)


def _picked(program, widths, B, dtype, k=2, sgd=False, **env):
    out = host_hip.run(program, "-".join(map(str, widths)), B, dtype, k, *(["sgd"] if sgd else []), **env).splitlines()
    return lambda what: [line.split(" ", 1)[1] for line in out if line.startswith(what + " ")]


def _routes(program, widths, B, dtype, k=2, sgd=False, **env):
    pick = _picked(program, widths, B, dtype, k, sgd, **env)
    return pick("forward"), pick("backward"), int(pick("noalloc")[0])


OK, UNSUPPORTED = 0, 5


@pytest.mark.parametrize("N,B,dtype,want", [
    # 128 x 128 tiles split to at most 512 workgroups: 8 MiB exactly, and one row of tiles more
    (2048, 128, "bf16", OK), (2048, 136, "bf16", UNSUPPORTED),
    (512, 256, "f32", OK), (4096, 256, "f32", UNSUPPORTED),
    (1600, 128, "f32", OK), (16384, 512, "f32", OK),                  # (the last: too many tiles for a split)
    # bf16 nets of 64 tiles of 256 x 256 and more, and the wide ones below that: the split of 256 x 256 tiles
    (1856, 4096, "bf16", OK), (2624, 3000, "bf16", OK), (3904, 2048, "bf16", OK),
    (8192, 48, "bf16", OK), (8000, 64, "bf16", OK), (16384, 32, "bf16", OK),
    (8192, 96, "bf16", UNSUPPORTED), (5120, 200, "bf16", UNSUPPORTED), (6144, 48, "bf16", UNSUPPORTED),
    (5120, 1536, "bf16", UNSUPPORTED),
    # (neither)
    (8320, 40, "bf16", UNSUPPORTED), (2048, 1024, "bf16", UNSUPPORTED),
    (8192, 1, "f32", OK), (16384, 1, "f32", UNSUPPORTED),             # single sample: row-block partial sums
])
def test_nets_served_without_allocation(program, N, B, dtype, want):
    assert _routes(program, [N] * 4, B, dtype)[2] == want


@pytest.mark.parametrize("N,B,dtype,mt,nt", [
    (9216, 32, "bf16", 2, 4),                                  # one turn of the compute units
    (8256, 33, "bf16", 4, 4), (9216, 48, "bf16", 4, 4),        # 4 x 4 blocks, one of them past the minibatch: still one turn
    (16384, 48, "f32", 4, 4),
])
def test_tile_of_a_direct_product(program, N, B, dtype, mt, nt):
    forward, backward, _ = _routes(program, [N] * 4, B, dtype, LF_GEMM_BIG="0")
    type_ = {"f32": "f", "bf16": "DF16b"}[dtype]
    assert len(forward) == 3 and all(f"k_forward_tileI{type_}Li{mt}ELi{nt}E" in name for name in forward)
    assert sum(f"k_backward_stepI{type_}Li{mt}ELi{nt}E" in name for name in backward) == 2


def test_tile_of_a_direct_forward_product_in_one_turn(program):
    forward, _, _ = _routes(program, [8192] * 4, 40, "bf16", LF_GEMM_BIG="0")
    assert len(forward) == 3 and all("k_forward_tileIDF16bLi2ELi4E" in name for name in forward)


@pytest.mark.parametrize("widths,B,dtype,want", [
    # (tile in 16 x 16 blocks, split over workgroups) of the chain steps, top layer first
    ([1536] * 4, 8, "bf16", [(1, 2, True)] * 2), ([2048] * 4, 32, "bf16", [(2, 2, True)] * 2),
    ([1536] * 4, 8, "f32", [(1, 2, True)] * 2), ([3072] * 4, 30, "f32", [(2, 4, True)] * 2),
    # the launch's workgroups would be a turn more
    ([1280] * 4, 8, "bf16", [(1, 2, False)] * 2), ([1600] * 4, 8, "bf16", [(1, 2, False)] * 2),
    ([1920] * 4, 24, "bf16", [(1, 2, False)] * 2),
    ([1280] * 4, 8, "f32", [(1, 1, False)] * 2), ([1920] * 4, 16, "f32", [(1, 1, False)] * 2),
    # contractions that are short beside the width, and long ones
    ([2048, 4096, 1024, 4096, 2048], 64, "bf16", [(2, 2, False), (1, 2, False), (2, 2, False)]),
    ([2048, 4096, 3072, 4096, 2048], 64, "bf16", [(2, 2, False), (2, 4, True), (2, 4, True)]),
    ([1024, 8192, 2048, 8192], 8, "bf16", [(1, 2, True), (1, 2, False)]),
    ([1024, 4096, 1024, 4096], 8, "f32", [(1, 2, True), (1, 1, False)]),
    ([1536, 2048, 1536, 2048], 8, "f32", [(1, 1, False), (1, 4, True)]),
    ([2048, 4096, 2048, 4096], 8, "bf16", [(1, 2, True), (1, 4, True)]),
    # a width is cut as its neighbours are
    *[([n] * 3, B, "bf16", [(4, 4, True)]) for n in (4104, 8128, 8136, 8192) for B in (33, 40, 48, 64)],
    *[([n] * 3, 64, "bf16", [(2, 4, True)]) for n in (3072, 4088, 4096)],
    *[([n] * 3, 8, "bf16", [(1, 4, True)]) for n in (2056, 3072, 8192)],
    # where the gradients beside it set the pace
    ([4608] * 3, 64, "f32", [(2, 4, False)]), ([4608] * 3, 40, "f32", [(4, 4, True)]), ([5632] * 3, 40, "f32", [(2, 4, False)]),
])
def test_chain_steps_are_split_where_that_pays(program, widths, B, dtype, want):
    _, backward, _ = _routes(program, widths, B, dtype, LF_GEMM_BIG="0")
    steps = [name for name in backward if "k_backward_step" in name][:len(want)]
    type_ = {"f32": "f", "bf16": "DF16b"}[dtype]
    got = []
    for name in steps:
        mt, nt, split = re.search(rf"k_backward_stepI{type_}Li(\d)ELi(\d)ELi\dELb[01]ELb([01])E", name).groups()
        got.append((int(mt), int(nt), split == "1"))
    assert got == want


@pytest.mark.parametrize("widths,B,dtype,want", [
    ((64, 3076, 3076, 260), 64, "f32", "IfLi2ELi4ELi2ELb1ELb1E"), ((64, 4100, 4100, 200), 52, "f32", "IfLi4ELi4ELi2ELb1ELb1E"),
    ((264, 1024, 1024, 260), 32, "f32", "IfLi1ELi1ELi2ELb0ELb0E"), ((64, 3072, 3072, 256), 64, "bf16", "IDF16bLi2ELi4ELi2ELb0ELb1E"),
    ((64, 1024, 1024, 256), 8, "bf16", "IDF16bLi1ELi2ELi2ELb0ELb1E"),
])
def test_descent_step_beside_a_chain_step_of_other_widths(program, widths, B, dtype, want):
    """The last chain step, beside which layer 4's descent step rides."""
    _, backward, _ = _routes(program, widths, B, dtype, sgd=True, LF_GEMM_BIG="0")
    assert f"k_backward_step{want}" in [name for name in backward if "k_backward_step" in name][1]


@pytest.mark.parametrize("widths,rows,streamed", [
    ([6000] * 3, 1, False), ([5000] * 4, 1, False), ([9000] * 2, 1, True), ([9600] * 2, 1, True),      # 275, 286, 309, 352 MB
    ([3000, 3004] * 4, 2, False), ([3000, 3004] * 6, 2, True),
])
def test_weights_beyond_the_cache_are_streamed_by_the_forward_product(program, widths, rows, streamed):
    forward, _, _ = _routes(program, widths, 1, "f32", k=1)
    assert forward and all(f"k_fwd_gemvILi{rows}ELb{int(streamed)}E" in name for name in forward)


# us a layer, (direct, wide-net kernels), measured at L = 6 .. 8, k = 4: the choice is to be the faster side
@pytest.mark.parametrize("N,B,forward,backward", [
    (256, 32768, (51, 26), (263, 537)), (1024, 512, (6.4, 16.8), (11.8, 28.3)), (1024, 4096, (27, 34), (69, 82)),
    (1536, 2048, (26, 30), (76, 54)), (2048, 128, (6.3, 17.3), (11.4, 28.4)), (2048, 1024, (17, 31), (35, 41)),
    (2048, 4096, (80, 52), (155, 90)), (2056, 1800, (58, 47), (110, 64)), (2560, 1024, (31, 48), (63, 54)),
    (3072, 384, (21, 26), (37, 41)), (3072, 768, (32, 46), (62, 49)), (3072, 2048, (85, 71), (178, 91)),
    (3584, 1024, (48, 65), (112, 80)), (4096, 8, (7.6, 17.2), (18.8, 33.3)), (4096, 128, (12, 22), (32, 38)),
    (4096, 512, (28, 37), (72, 53)), (4096, 1024, (59, 50), (124, 77)), (4360, 200, (34, 34), (60, 49)),
    (4608, 320, (36, 46), (60, 52)), (5016, 240, (42, 54), (72, 62)), (5120, 64, (21, 31), (27, 40)),
    (5120, 256, (41, 53), (62, 54)), (5120, 2048, (230, 139), (428, 180)), (5384, 700, (98, 85), (190, 114)),
    (6144, 256, (50, 58), (90, 74)), (6144, 512, (67, 70), (146, 99)), (7000, 150, (71, 55), (102, 93)),
    (7168, 256, (57, 67), (120, 92)), (8192, 32, (31, 36), (70, 75)), (8192, 192, (67, 49), (118, 89)),
    (8192, 512, (108, 78), (258, 148)), (10240, 128, (97, 79), (157, 115)), (12288, 384, (216, 166), (444, 256)),
    (16384, 8, (99, 139), (259, 261)), (16384, 256, (238, 179), (595, 312)),
    (6144, 128, (35, 44), (63, 56)), (6656, 80, (32, 40), (59, 64)), (7168, 96, (35, 45), (69, 73)),
])
def test_bf16_nets_take_the_faster_kernels(program, N, B, forward, backward):
    """(sides within 6 % of each other are as good; L = 6)"""
    fwd, bwd, _ = _routes(program, [N] * 6, B, "bf16")
    for names, (direct, wide), direct_kernel in ((fwd, forward, "k_forward_tile"), (bwd, backward, "k_backward_step")):
        took_direct = any(direct_kernel in name for name in names)
        assert took_direct != any("k_gemm_big" in name for name in names)
        assert (direct if took_direct else wide) <= 1.06 * min(direct, wide), (took_direct, direct, wide)


@pytest.mark.parametrize("widths,B,fwd_direct,bwd_direct", [
    ([8192] + [1024] * 7, 256, True, True),               # one wide layer decides nothing: 6.5 / 16 us forward, 9.6 / 26 backward
    ([2048] + [256] * 5, 2048, True, True),               # 7.6 / 22, 19 / 41
    ([4096, 11008, 4096, 11008, 4096], 512, False, False),      # 82 / 79, 179 / 111
])
def test_all_layers_have_a_say_in_the_choice(program, widths, B, fwd_direct, bwd_direct):
    fwd, bwd, _ = _routes(program, widths, B, "bf16")
    assert all("k_forward_tile" in name for name in fwd) if fwd_direct else not any("k_forward_tile" in name for name in fwd)
    assert any("k_backward_step" in name for name in bwd) == bwd_direct


def test_fp32_nets_take_the_direct_kernels(program):
    for N, B in ((64, 2), (2048, 2048), (8192, 1024)):
        fwd, bwd, _ = _routes(program, [N] * 4, B, "f32")
        assert all("k_forward_tile" in name for name in fwd) and sum("k_backward_step" in name for name in bwd) == 3


@pytest.mark.parametrize("widths,streamed", [([4096] * 4, 3), ([4104] * 4, 0), ([4096, 4104, 4096, 4096], 2)])
def test_streamed_gradients_have_rows_of_whole_lines(program, widths, streamed):
    """One product a layer: the streamed kernel where n_prev is a multiple of 32, else a workgroup per tile."""
    _, bwd, _ = _routes(program, widths, 1024, "bf16")
    grads = [name for name in bwd if "k_grad_stream" in name or "k_gemm_bigILb1ELb1E" in name]
    assert len(grads) == 3 and sum("k_grad_stream" in name for name in grads) == streamed


@pytest.mark.parametrize("N,dtype", [(256, "f32"), (512, "bf16")])
def test_each_pass_of_a_small_net_prepares_what_its_workgroups_exchange(program, N, dtype):
    """The workspace may have held anything since the last pass: its counters and words are cleared in front of every
    forward pass, the first as the next."""
    pick = _picked(program, [N] * 6, 32, dtype, LF_CLUSTER="1")
    for names in (pick("forward"), pick("again")):
        assert len(names) == 2 and "k_cluster_state" in names[0] and "k_clusterI" in names[1]
    assert "k_clusterI" in pick("backward")[0] and "k_all_gradients" in pick("backward")[1]


# us a pass forward / backward, measured: by a launch a layer, and by one for all (the forward pass with its preparation)
@pytest.mark.parametrize("widths,B,dtype,layers,one", [
    ([64] * 8, 32, "f32", (19, 29), (12, 15)), ([256] * 8, 32, "f32", (21, 31), (17, 21)), ([256] * 8, 300, "f32", (27, 43), (22, 36)),
    ([256] * 8, 1024, "f32", (37, 75), (47, 70)), ([256] * 8, 4096, "f32", (114, 234), (187, 265)), ([512] * 10, 128, "f32", (34, 57), (34, 47)),
    ([512] * 8, 256, "f32", (34, 60), (38, 67)), ([512] * 8, 1024, "f32", (62, 112), (124, 226)), ([384] * 8, 512, "f32", (39, 60), (43, 72)),
    ([64] * 16, 4096, "f32", (117, 416), (80, 101)), ([64] * 8, 16384, "f32", (247, 748), (232, 293)),
    ([256] * 8, 64, "bf16", (21, 31), (15, 20)), ([512] * 8, 64, "bf16", (22, 32), (19, 30)), ([512] * 16, 256, "bf16", (55, 91), (36, 56)),
    ([512] * 5, 384, "bf16", (17, 26), (19, 44)), ([704] * 5, 384, "bf16", (23, 38), (26, 70)), ([704] * 8, 384, "bf16", (40, 66), (41, 88)),
    ([768] * 16, 64, "bf16", (49, 72), (46, 70)), ([768] * 16, 65, "bf16", (49, 81), (46, 70)), ([896] * 16, 128, "bf16", (62, 152), (57, 90)),
    ([1024] * 8, 32, "bf16", (24, 47), (35, 52)), ([1024] * 8, 256, "bf16", (35, 59), (46, 90)), ([256] * 5, 32640, "bf16", (106, 947), (866, 1243)),
    ([128] * 16, 4096, "bf16", (132, 467), (83, 145)),
    # unequal widths: the widest contraction of a launch decides what each of its steps takes
    ([64] * 4 + [512] + [64] * 3, 512, "f32", (23, 50), (28, 32)), ([512] + [64] * 7, 512, "f32", (21, 48), (23, 19)),
    ([64] * 7 + [512], 32, "f32", (20, 30), (15, 28)), ([64, 512] * 4, 512, "f32", (31, 54), (45, 54)), ([300, 44, 76, 512, 308], 448, "f32", (17, 33), (25, 47)),
    ([64, 1024] * 4, 512, "bf16", (31, 47), (49, 70)), ([784] + [256] * 6 + [16], 32, "bf16", (21, 31), (22, 18)),
    ([64] * 4 + [512] + [64] * 3, 32, "f32", (20, 30), (22, 24)), ([192] * 5 + [848, 192], 1030, "bf16", (34, 56), (45, 92)), ([160, 56, 56, 136, 832], 10, "bf16", (13, 19), (12, 28)),
])
def test_small_nets_take_the_faster_kernels(program, widths, B, dtype, layers, one):
    """The choice is no more than 4 % off the best of: a launch a layer, one for the chain alone (and its preparation), one a direction."""
    forward, backward, _ = _routes(program, widths, B, dtype)
    here = [any("k_clusterI" in name for name in names) for names in (forward, backward)]
    assert any("k_all_gradients" in name for name in backward) == here[1]
    times = {(False, False): sum(layers), (False, True): layers[0] + one[1] + 1.8, (True, True): sum(one)}
    assert times[tuple(here)] <= 1.04 * min(times.values()), (here, times)
    prepared = sum("k_cluster_state" in name for name in forward), sum("k_cluster_state" in name for name in backward)
    assert prepared == (here[0], here[1] and not here[0])


@pytest.mark.parametrize("widths,dtype", [([64] * 4, "f32"), ([516] + [64] * 9, "f32"), ([64] * 9 + [1032], "bf16")])
def test_few_layers_and_wide_ones_take_a_launch_a_layer(program, widths, dtype):
    forward, backward, _ = _routes(program, widths, 32, dtype)
    assert not any("k_cluster" in name for name in forward + backward)


@pytest.mark.parametrize("choice,kernels", [("0", ("k_forward_tile", "k_backward_step")), ("1", ("k_gemm_big", "k_gemm_big"))])
def test_the_forced_choice_of_kernels_holds_for_small_nets(program, choice, kernels):
    forward, backward, noalloc = _routes(program, [256] * 8, 32, "bf16", LF_GEMM_BIG=choice)
    for names, kernel in zip((forward, backward), kernels):
        assert any(kernel in name for name in names)
        assert not any("k_cluster" in name or "k_all_gradients" in name for name in names)
    assert noalloc == OK


# argv: how the lost pass is found out.  A wait of a small net's kernels that gave up has raised the pinned word.
LOST = r"""
int main(int, char** argv) {
    lf_net* net = make({256, 256, 256, 256, 256, 256}, 32, LF_F32, std::string(argv[1]) == "streams" ? LF_SCHED_STREAMS : LF_SCHED_AUTO);
    const std::string by = argv[1];
    CHECK(lf_forward(net, some_input, &caller_1) == LF_OK);
    CHECK((created == 0) == (by == "streams"));          // (that schedule's forward pass allocates nothing)
    CHECK(lf_backward_leapfrog(net, some_input, 2, &caller_1) == LF_OK);
    CHECK(pinned != nullptr);
    if (!pinned) return 1;
    *(int*)pinned = (4 << 24) | (3 << 10) | 7;
    lf_status st = by == "forward" || by == "streams" ? lf_forward(net, some_input, &caller_1)
                   : by == "backward" ? lf_backward_leapfrog(net, some_input, 1, &caller_1)
                   : by == "noalloc" ? lf_backward_leapfrog_noalloc(net, some_input, 1, &caller_1) : lf_grads(net, 2, nullptr, nullptr);
    CHECK(st == LF_EHIP);
    std::printf("%s\n", lf_last_error(net));
    CHECK(lf_backward_leapfrog(net, some_input, 1, &caller_1) == LF_ESTATE);
    launched.clear();
    CHECK(lf_forward(net, some_input, &caller_1) == LF_OK);
    CHECK(lf_backward_leapfrog(net, some_input, 2, &caller_1) == LF_OK);
    CHECK(lf_backward_leapfrog_noalloc(net, some_input, 1, &caller_1) == LF_OK);
    CHECK(!launched.empty());
    for (const std::string& s : launched) CHECK(s.find("k_cluster") == std::string::npos && s.find("k_all_gradients") == std::string::npos);
    lf_destroy(net);
    return failures != 0;
}
"""


@pytest.mark.parametrize("by", ["forward", "backward", "noalloc", "grads", "streams"])
def test_a_small_net_that_lost_a_pass_says_so_and_does_without_these_kernels(tmp_path, by):
    out = host_hip.run(host_hip.build(tmp_path, LOST), by, LF_CLUSTER="1")
    assert "layer 3, workgroup 7" in out and "run lf_forward again" in out


# Every handle has a pinned word of its own, from one page for 1024 of them, and gives it back; without pinned memory the passes
# of small nets run all the same.
WORDS = r"""
#include <algorithm>
int main() {
    std::vector<lf_net*> nets;
    std::vector<void*> words;
    auto add = [&]() {
        nets.push_back(make({64, 64, 64, 64, 64, 64}, 8, LF_F32, LF_SCHED_AUTO));
        pinned_word = nullptr;
        CHECK(lf_forward(nets.back(), some_input, &caller_1) == LF_OK);
        CHECK(pinned_word != nullptr && std::find(words.begin(), words.end(), pinned_word) == words.end());
        words.push_back(pinned_word);
    };
    for (int i = 0; i < 1030; ++i) add();
    CHECK(created == 1 + 6);
    for (int i = 0; i < 500; ++i) {                       // the ones in the middle go
        lf_destroy(nets[100]);
        nets.erase(nets.begin() + 100);
        words.erase(words.begin() + 100);
    }
    for (int i = 0; i < 500; ++i) add();
    CHECK(created == 1 + 6);
    for (lf_net* net : nets) lf_destroy(net);
    nets.clear(); words.clear();
    for (int i = 0; i < 1024; ++i) add();
    CHECK(created == 1 + 6);
    no_pinned_memory = true;
    lf_net* net = make({64, 64, 64, 64, 64, 64}, 8, LF_F32, LF_SCHED_AUTO);
    CHECK(lf_forward(net, some_input, &caller_1) == LF_OK);
    CHECK(lf_backward_leapfrog(net, some_input, 1, &caller_1) == LF_OK);
    lf_destroy(net);
    for (lf_net* n : nets) lf_destroy(n);
    return failures != 0;
}
"""


def test_handles_share_a_page_of_pinned_words(tmp_path):
    host_hip.run(host_hip.build(tmp_path, WORDS), LF_CLUSTER="1")
