"""Which unit (request, v-head) a workgroup of kvb_direct takes, from the functions of csrc/kvb_device.h run on the host."""
import os
import subprocess

import numpy as np
import pytest

from paper_2605_19049_amd import build

SRC = r"""
#include "kvb_device.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char **argv)
{
    const int blocks = atoi(argv[1]), deal = kvb_impl::deal_of(blocks, atoi(argv[2]));
    for (int x = 0; x < blocks; ++x)
        printf("%d\n", kvb_impl::dealt_unit(x, deal));
}
"""


@pytest.fixture(scope="module")
def units(tmp_path_factory):
    d = tmp_path_factory.mktemp("dealing")
    src, exe = os.path.join(d, "deal.hip"), os.path.join(d, "deal")
    with open(src, "w") as f:
        f.write(SRC)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc] + build.HIPCC_FLAGS + ["-o", exe, src], check=True, stderr=subprocess.DEVNULL)

    def run(blocks, r):
        return np.array(subprocess.run([exe, str(blocks), str(r)], check=True, stdout=subprocess.PIPE, text=True).stdout.split(), int)
    return run


@pytest.mark.parametrize("B, Hk, Hv", [(64, 16, 32), (13, 4, 8), (5, 4, 16), (7, 2, 16), (3, 8, 24), (5, 3, 9), (1, 1, 1), (1, 8, 8), (500, 16, 32), (255, 4, 8), (101, 4, 16), (2, 1, 8), (300000, 1, 32)])
def test_dealing(units, B, Hk, Hv):
    """Every unit is taken once.  Where the qk-heads divide by 8, and from 1024 units on, the v-heads of a qk-head share an
    XCD (workgroup id modulo 8), all but those of fewer than 8 qk-heads, and every XCD has as many qk-heads."""
    blocks, r = B * Hv, Hv // Hk
    u = units(blocks, r)
    assert np.array_equal(np.sort(u), np.arange(blocks))
    xcd = np.empty(blocks, int)
    xcd[u] = np.arange(blocks) % 8
    split = (xcd.reshape(B * Hk, r) != xcd[::r, None]).any(1).sum()
    if B * Hk % 8 and blocks < 1024:
        return
    assert split <= B * Hk % 8, split
    whole = xcd.reshape(B * Hk, r)[:B * Hk // 8 * 8, 0]
    assert np.ptp(np.bincount(whole, minlength=8)) == 0
