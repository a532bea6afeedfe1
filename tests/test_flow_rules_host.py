"""Which layers stream in persistent blocks (csrc/ffn_rules.hpp, compiled for the host): those of tests/test_gpu_flow.py do, the batches
they are compared with do not."""
import subprocess

import numpy as np
import pytest

import test_gpu_dispatch as dispatch
from paper_2512_07710_amd.build import CSRC, HIPCC, ROOT

EDGE_ROWS = np.array([1, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81, 96, 97, 0, 5, 200, 15, 2, 31, 47, 63, 79, 95, 100, 8, 129])
# d, E, k, F, quarters of EDGE_ROWS: four K blocks, the fewest; odd widths (the down projection's last unit half empty); one block with
# several units and with none behind; more K blocks than lanes; two experts a token
LAYERS = {"fewest-k-blocks": (512, 40, 1, 512, 4), "odd-widths": (640, 30, 1, 640, 4), "few-rows": (1152, 60, 1, 512, 1),
          "wide": (8448, 40, 1, 512, 2), "two-a-token": (768, 90, 2, 512, 4), "many-units": (512, 120, 1, 896, 2)}
PROGRAM = r"""
#include "ffn_rules.hpp"
#include <cstdio>
using namespace moe355;
int main() {
    moe_dims D{};
    while (scanf("%d %d %d %d %d", &D.T, &D.d, &D.E, &D.k, &D.F) == 5) printf("%d%d\n", gate_up_flows(&D), down_flows(&D));
    return 0;
}
"""


@pytest.fixture(scope="module")
def flows(tmp_path_factory):
    d = tmp_path_factory.mktemp("flow_rules")
    (d / "rules.hip").write_text(PROGRAM)
    subprocess.run([HIPCC, "--cuda-host-only", "-O2", "-std=c++17", "-I", CSRC, "-I", ROOT + "/include", str(d / "rules.hip"), "-o",
                    str(d / "rules")], check=True, capture_output=True)

    def ask(*shapes):
        text = "\n".join(" ".join(map(str, s)) for s in shapes)
        return subprocess.run([str(d / "rules")], input=text, check=True, capture_output=True, text=True).stdout.split()
    return ask


def _tokens(E, k, scale):
    counts = np.resize(EDGE_ROWS, E) * scale // 4
    return int(counts.sum()) if k == 1 else int(((counts + 1) // 2).sum())


def test_the_layers_of_the_gpu_test_flow_and_their_references_do_not(flows):
    met = set()
    for d, E, k, F, scale in LAYERS.values():
        T = _tokens(E, k, scale)
        here, big = flows((T, d, E, k, F), (T + 97 * (E + k), d, E + k, k, F))
        assert here[0] == "1" and big == "00", (d, E, k, F)
        met.add(here)
    assert met == {"10", "11"}


def test_the_graph_tests_layers_are_what_their_names_say(flows):
    assert dict(zip(dispatch.GRAPH_LAYERS, flows(*dispatch.GRAPH_LAYERS.values()))) == {
        "streaming": "00", "chosen-on-device": "00", "persistent-blocks": "10", "persistent-blocks-down": "11"}


def test_what_the_persistent_kernel_cannot_take_is_not_given_to_it(flows):
    """Fewer than four K blocks in either projection, more than 128; more rows per expert than a tile on the mean; no rows."""
    T, E, k = 1500, 64, 1
    asked = flows((T, 512, E, k, 512), (T, 384, E, k, 512), (T, 512, E, k, 384), (T, 128 * 128, E, k, 512), (T, 129 * 128, E, k, 512),
                  (96 * E + 1, 512, E, k, 512), (0, 512, E, k, 512))
    assert [a[0] for a in asked] == ["1", "0", "0", "1", "0", "0", "0"]
    assert all(a[0] == "1" or a[1] == "0" for a in asked)


def test_few_rows_of_a_single_round_stay_with_the_streaming_kernel(flows):
    """About one row per expert: a skewed log meets far fewer experts than an even one, which would leave a single round half empty."""
    assert flows((63, 4480, 69, 1, 640), (256, 4096, 64, 6, 1408)) == ["00", "10"]
