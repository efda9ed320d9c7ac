"""How the visibility route cuts a call into launches (csrc/fx_tables.h, plain C++):
the workspace it asks for and the passes over time, over the accepted range."""
import itertools
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1510_08318_amd", "csrc")
GIB = 1 << 30
MAIN = """
#include <cstdio>
#include "fx_tables.h"
int main() {
  int ci4, n_ant, n_chan;
  long long n_time, fixed;
  while (std::scanf("%d %d %d %lld %lld", &ci4, &n_ant, &n_chan, &n_time, &fixed) == 5) {
    const moff::FxChunks f = moff::fx_chunks(ci4 != 0, n_ant, n_chan, n_time, static_cast<size_t>(fixed));
    std::printf("%d %lld %zu %zu %zu %zu\\n", f.channels, static_cast<long long>(f.pass), f.samples, f.sums, f.per_channel,
                moff::fx_plane_bytes(ci4 != 0, n_ant, f.pass));
  }
}
"""


@pytest.fixture(scope="module")
def chunks(tmp_path_factory):
    d = tmp_path_factory.mktemp("fx")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "main")], check=True)

    def run(rows):
        text = "\n".join(" ".join(str(int(x)) for x in r) for r in rows)
        out = subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    return run


def test_chunks_over_the_accepted_range(chunks):
    rows = [(ci4, a, c, t, 8 * a * a + extra)
            for ci4, a, c, t, extra in itertools.product(
                (0, 1), (2, 64, 65, 350, 1024, 2900, 3340, 3341, 3400, 4000), (1, 5, 8, 9, 300),
                (1, 33, 1000, 20000, 400003, 1 << 24), (1 << 10, 9 << 20))]
    for (ci4, a, c, t, fixed), (chan, pass_, samples, sums, per, plane) in zip(rows, chunks(rows)):
        label = (ci4, a, c, t, fixed)
        visibilities = 8 * a * a
        few = min(c, 8)
        assert 1 <= pass_ <= t and samples == plane, label
        assert per >= fixed + samples + sums and per % 256 == 0, label
        assert few <= chan <= min(c, 65535), label                       # every XCD has a channel
        assert chan * per <= max(2 * GIB, few * (fixed + 24 * a * a + 2 * (24576 + 256) * ((a + 63) // 64))), label
        if pass_ < t:
            assert sums == 16 * a * a and pass_ % (64 if ci4 else 32) == 0, label
            # the sums that a pass reads and writes are at most four times its samples
            assert samples >= 0.9 * visibilities, label
            assert (fixed + plane * -(-t // pass_)) * few > 2 * GIB * 0.9, label   # one pass would not have fit
        else:
            assert sums == 0, label


def test_no_pass_of_a_single_step(chunks):
    """4000 antennas, eight channels, 3000 complex64 samples: two passes, not 94."""
    (chan, pass_, *_), = chunks([(0, 4000, 8, 3000, 8 * 4000 ** 2 + (1 << 20))])
    assert chan == 8 and -(-3000 // pass_) <= 2
