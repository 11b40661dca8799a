"""Which kernels a net's passes launch, and which nets lf_backward_leapfrog_noalloc serves, from the calls the library makes
on the host (no kernel runs)."""
import pytest

from tests import host_hip

# argv: widths, B, dtype, k.  Prints the kernels of a forward pass, of a backward pass, and the status of the
# no-alloc backward pass.
MAIN = r"""
#include <sstream>
int main(int, char** argv) {
    std::vector<int> n;
    std::stringstream widths(argv[1]);
    for (std::string w; std::getline(widths, w, '-');) n.push_back(std::atoi(w.c_str()));
    lf_net* net = make(n, std::atoi(argv[2]), argv[3][0] == 'b' ? LF_BF16 : LF_F32, LF_SCHED_AUTO);
    auto print = [&](const char* what) {
        for (const std::string& s : launched) std::printf("%s %s\n", what, s.c_str());
        launched.clear();
    };
    CHECK(lf_forward(net, some_input, &caller_1) == LF_OK);
    print("forward");
    CHECK(lf_backward_leapfrog(net, some_input, std::atoi(argv[4]), &caller_1) == LF_OK);
    print("backward");
    std::printf("noalloc %d\n", (int)lf_backward_leapfrog_noalloc(net, some_input, 1, &caller_1));
    lf_destroy(net);
    return failures != 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return host_hip.build(tmp_path_factory.mktemp("routes"), MAIN)


def _routes(program, widths, B, dtype, k=2, **env):
    out = host_hip.run(program, "-".join(map(str, widths)), B, dtype, k, **env).splitlines()
    pick = lambda what: [line.split(" ", 1)[1] for line in out if line.startswith(what + " ")]  # noqa: E731
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
    (8192, 40, "bf16", 2, 4), (9216, 32, "bf16", 2, 4),        # one turn of the compute units
    (8256, 33, "bf16", 4, 4), (9216, 48, "bf16", 4, 4),        # 4 x 4 blocks, one of them past the minibatch: still one turn
    (16384, 48, "f32", 4, 4),
])
def test_tile_of_a_direct_product(program, N, B, dtype, mt, nt):
    forward, backward, _ = _routes(program, [N] * 4, B, dtype, LF_GEMM_BIG="0")
    type_ = {"f32": "f", "bf16": "DF16b"}[dtype]
    assert len(forward) == 3 and all(f"k_forward_tileI{type_}Li{mt}ELi{nt}E" in name for name in forward)
    assert sum(f"k_backward_stepI{type_}Li{mt}ELi{nt}E" in name for name in backward) == 2
