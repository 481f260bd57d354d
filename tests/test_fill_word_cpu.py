"""What a wave makes of a fill word that other workgroups are changing, from the functions of csrc/kvb_device.h run on
the host over every state that the word goes through."""
import os
import subprocess

import pytest

from paper_2605_19049_amd import build

SRC = r"""
#include "kvb_device.h"
#include <cstdio>
#include <cstdlib>
using namespace kvb_impl;
// Every set of shares that can be missing: `others` of the workgroups and, or not, the first.  Returns the number of
// wrong readings and wrong final words.
static long long states(int nwg, int old, int change, int folded, bool commit)
{
    long long bad = 0;
    for (int others = 0; others < nwg; ++others)
        for (int first = 0; first < 2; ++first) {
            uint32_t w = (uint32_t)old;
            for (int i = 0; i < others; ++i)
                w += (uint32_t)fill_share(false, nwg, change);
            if (first)
                w += (uint32_t)fill_share(true, nwg, change);
            if (first && others == nwg - 1)
                bad += w != (uint32_t)(old + change);
            else
                bad += (commit ? fill_before_commit((int)w, change) : fill_before((int)w, folded)) != old;
        }
    return bad;
}
int main(int argc, char **argv)
{
    const int nwg = atoi(argv[1]);
    long long bad = 0;
    if (nwg > 4096) {   // the words at the ends of what bits 16.. can count: shares in, of the others, and of the first or not
        for (int old = 0; old <= 128; old += 64)
            for (int change = -old; change <= 8; ++change)
                for (int others : {0, 1, nwg - 2, nwg - 1}) {
                    const uint32_t w = (uint32_t)old + (uint32_t)others * (uint32_t)fill_share(false, nwg, change);
                    const uint32_t all = w + (uint32_t)fill_share(true, nwg, change);
                    bad += (int)w < 0 || ((int)w & FILL_MASK) != old;
                    bad += others == nwg - 1 ? all != (uint32_t)(old + change) : (int)all >= 0 || ((int)all & FILL_MASK) != old + change;
                }
        printf("%lld\n", bad);
        return 0;
    }
    for (int old = 0; old <= 128; old += nwg > 1000 ? 127 : 1) {
        bad += states(nwg, old, 1, 16, false);          // a token was appended (whatever the threshold is)
        bad += states(nwg, old, -old, old, false);      // and the buffer folded, at threshold old + 1
        for (int acc = 1; acc <= 8; ++acc)
            bad += states(nwg, old, acc, 0, true);      // accepted records were committed
    }
    printf("%lld\n", bad);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("fill_word")
    src, exe = os.path.join(d, "fill.hip"), os.path.join(d, "fill")
    with open(src, "w") as f:
        f.write(SRC)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc] + build.HIPCC_FLAGS + ["-o", exe, src], check=True, stderr=subprocess.DEVNULL)
    return exe


@pytest.mark.parametrize("nwg", [1, 2, 3, 32, 255, 4096, 32768])
def test_every_state_of_the_word(program, nwg):
    """A reading gives the old fill until the last share is in; then the word is the new fill."""
    assert int(subprocess.run([program, str(nwg)], check=True, stdout=subprocess.PIPE, text=True).stdout) == 0
