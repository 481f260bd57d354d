"""Which unit (request, v-head) a workgroup of kvb_direct takes, in which launches the requests are sorted, and which rows the
lanes read, from the functions of csrc/kvb_device.h run on the host."""
import os
import subprocess

import numpy as np
import pytest

from paper_2605_19049_amd import build

SRC = r"""
#include "kvb_device.h"
#include <cstdio>
#include <cstdlib>
#include <utility>
int main(int argc, char **argv)
{
    if (argc == 1) {   // d, input type, units, longest context of every launch that sorts
        for (int d : {32, 64, 128})
            for (int type : {KVB_F32, KVB_BF16, KVB_F16})
                for (int blocks = 1; blocks < 20000; blocks += blocks < 3000 ? 1 : 997)
                    for (int Lmax = 1; Lmax <= 128; ++Lmax)
                        if (kvb_impl::longest_first(blocks, Lmax, d, type))
                            printf("%d %d %d %d\n", d, type, blocks, Lmax);
        return 0;
    }
    if (argc == 2) {   // wrong row offsets for a number of heads of 128 16-bit elements
        const uint32_t stride = (uint32_t)atoi(argv[1]) * 256u;
        int bad = 0;
        for (int left = 0; left < 128; ++left)
            for (int row = 0; row < 16; ++row)
                bad += kvb_impl::row_of_16((uint32_t)row * stride, left, stride) != (uint32_t)(row < left ? row : left) * stride;
        printf("%d\n", bad);
        return 0;
    }
    if (argc == 4) {   // units of the kernels that share fill words, dealt from argv[3] units on
        const int n = atoi(argv[1]);
        const uint32_t word = (uint32_t)kvb_impl::unit_deal(n, atoi(argv[2]), atoi(argv[3]));
        for (int x = 0; x < n; ++x)
            printf("%d\n", kvb_impl::unit_of((uint32_t)x, word));
        return 0;
    }
    if (argc == 3 && atoi(argv[1]) == 0) {   // the rules that look at where the fill words lie
        if (atoi(argv[2]) == 0) {   // units to deal from: d, units, threshold, apart, of kvb_step_kernel (plain, streamed, kvb_verify), folds of 16 and of 17 records, a commit, others at 512
            for (int d : {32, 64, 128})
                for (int n : {1, 511, 512, 767, 768, 831, 832, 1023, 1024, 1535, 1536, 3839, 3840, 100000})
                    for (int threshold : {0, 1, 2, 3, 16})
                        for (int apart = 0; apart < 2; ++apart)
                            printf("%d %d %d %d %d %d %d %d %d %d %d\n", d, n, threshold, apart, kvb_impl::step_deals_from(d, n, threshold, false, true, apart),
                                   kvb_impl::step_deals_from(d, n, threshold, true, true, apart), kvb_impl::step_deals_from(d, n, threshold, false, false, apart),
                                   kvb_impl::fold_deals_from(d, n, false, threshold, 16, apart), kvb_impl::fold_deals_from(d, n, false, threshold, 17, apart),
                                   kvb_impl::fold_deals_from(d, n, true, threshold, 128, apart), kvb_impl::deals_from(512, apart));
            return 0;
        }
        // v-heads of a workgroup of kvb_decode without a state: d, fp32 inputs, heads, cap, requests, apart, answer
        for (int d : {32, 64, 128})
            for (int wide = 0; wide < 2; ++wide)
                for (auto [Hk, Hv] : {std::pair(1, 1), {1, 2}, {4, 4}, {3, 9}, {16, 32}, {1, 32768}, {1, 32769}, {16384, 65536}})
                    for (int cap : {16, 64, 65, 128})
                        for (int B : {1, 2, 3, 7, 8, 10, 11, 13, 36, 60, 96, 256, 320, 500})
                            for (int apart = 0; apart < 2; ++apart)
                                printf("%d %d %d %d %d %d %d %d\n", d, wide, Hk, Hv, cap, B, apart,
                                       kvb_impl::buffer_step_heads(d, wide, Hk, Hv, cap, B * Hv, apart));
        return 0;
    }
    const int blocks = atoi(argv[1]), deal = kvb_impl::deal_of(blocks, atoi(argv[2]));
    for (int x = 0; x < blocks; ++x)
        printf("%d\n", kvb_impl::dealt_unit(x, deal));
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("dealing")
    src, exe = os.path.join(d, "deal.hip"), os.path.join(d, "deal")
    with open(src, "w") as f:
        f.write(SRC)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc] + build.HIPCC_FLAGS + ["-o", exe, src], check=True, stderr=subprocess.DEVNULL)

    def run(*args):
        return np.array(subprocess.run([exe] + [str(a) for a in args], check=True, stdout=subprocess.PIPE, text=True).stdout.split(), int)
    return run


@pytest.mark.parametrize("B, Hk, Hv", [(64, 16, 32), (13, 4, 8), (5, 4, 16), (7, 2, 16), (3, 8, 24), (5, 3, 9), (1, 1, 1), (1, 8, 8), (500, 16, 32), (255, 4, 8), (101, 4, 16), (2, 1, 8), (300000, 1, 32)])
def test_dealing(program, B, Hk, Hv):
    """Every unit is taken once.  Where the qk-heads divide by 8, and from 1024 units on, the v-heads of a qk-head share an
    XCD (workgroup id modulo 8), all but those of fewer than 8 qk-heads, and every XCD has as many qk-heads."""
    blocks, r = B * Hv, Hv // Hk
    u = program(blocks, r)
    assert np.array_equal(np.sort(u), np.arange(blocks))
    xcd = np.empty(blocks, int)
    xcd[u] = np.arange(blocks) % 8
    split = (xcd.reshape(B * Hk, r) != xcd[::r, None]).any(1).sum()
    if B * Hk % 8 and blocks < 1024:
        return
    assert split <= B * Hk % 8, split
    whole = xcd.reshape(B * Hk, r)[:B * Hk // 8 * 8, 0]
    assert np.ptp(np.bincount(whole, minlength=8)) == 0


def test_no_sort_without_different_lengths(program):
    """Contexts of up to 16 tokens are all of one class of the sort, which would cost each workgroup a barrier and a scan for
    the order of the batch.  Longer ones: in launches of more than a round, and at most of a few."""
    d, _, blocks, Lmax = program().reshape(-1, 4).T
    assert Lmax.min() > 16
    short = Lmax <= 64
    assert blocks[short].min() >= 320 and blocks[short].max() <= 2560
    assert (d[blocks == blocks.max()] == 128).any() and blocks[~short].max() > 10000   # above 64 tokens without an upper line


@pytest.mark.parametrize("heads", [1, 32, 132104, 132105, 200000, 264207, 1000000])
def test_row_offsets(program, heads):
    """A row of 16, or the last one there is, also where the rows of a whole context leave 32 bits."""
    assert program(heads)[0] == 0


@pytest.mark.parametrize("B, Hk, r", [(64, 16, 2), (13, 4, 2), (1, 16, 2), (7, 2, 4), (5, 3, 3), (24, 3, 3), (16, 3, 3), (1, 1, 1), (1, 8, 1), (23, 16, 1), (500, 16, 2), (255, 4, 2), (3, 1, 16), (2, 8, 8)])
@pytest.mark.parametrize("least", [0, 512])
def test_units_of_shared_fill_words(program, B, Hk, r, least):
    """Every unit is taken once.  Dealt, where the qk-heads divide by 8, r is a power of two and the units are enough: the v-heads of
    a qk-head on one XCD (workgroup id modulo 8), consecutive qk-heads on consecutive ones; else whole eighths, or as they come."""
    n = B * Hk * r
    u = program(n, r, least)
    assert np.array_equal(np.sort(u), np.arange(n))
    xcd = np.empty(n, int)
    xcd[u] = np.arange(n) % 8
    if n >= least and r & (r - 1) == 0 and B * Hk % 8 == 0:
        assert np.array_equal(xcd, np.arange(n) // r % 8)
    elif n % 8 == 0:
        assert np.array_equal(xcd, np.arange(n) // (n // 8))
    else:
        assert np.array_equal(u, np.arange(n))


def test_which_launches_deal(program):
    """Where every step folds (or, streamed, every second) no unit is dealt, at d = 128 from 1024 units on; kvb_decode and the fold behind it are alike at any
    size, kvb_verify and the commit behind it too, but where every request folds, or nearly, at d = 128 and the state is no larger
    than the last-level cache.  With 32 fill words to a line only kvb_decode_flush at d = 128 and from 512 to 831 units deals."""
    rows = program(0, 0).reshape(-1, 11)
    assert len(rows) == 3 * 14 * 5 * 2
    never = 2 ** 31 - 1
    for d, n, threshold, apart, step, streamed, verify, fold, fold_long, commit, other in rows:
        large = d < 128 or n >= 1024
        for got, level in ((step, large and threshold == 1), (streamed, large and threshold in (1, 2))):   # (level: every step folds, or every second)
            if apart:
                assert got == (never if level else 512 if threshold else 0)
            else:
                assert got == (512 if d == 128 and threshold and n < 832 else never)
        if apart:
            cached = d == 128 and 768 <= n < 3840
            assert fold == (never if cached and threshold == 1 else 0) and fold_long == 0
            assert commit == (never if cached and (threshold == 1 or (threshold == 2 and n >= 1536)) else 512)
            assert other == 512 and (threshold or verify == 512)
        else:
            assert fold == fold_long == commit == other == never
    assert np.array_equal(program(2048, 2, never), np.arange(2048) % 8 * 256 + np.arange(2048) // 8)   # (eighths)


def test_heads_of_a_buffer_step(program):
    """Two v-heads a workgroup by the lines of each layout of the fill words; where one head has more workgroups a request than a
    word counts (2^15) and two do not, two are taken."""
    rows = program(0, 1).reshape(-1, 8)
    assert len(rows) == 3 * 2 * 8 * 4 * 14 * 2
    for d, wide, Hk, Hv, cap, B, apart, heads in rows:
        n, grouped = B * Hv, Hv > Hk
        if not apart:
            assert heads == (2 if grouped and n >= (256 if d == 128 else 96) else 1)
        else:
            assert heads == (2 if grouped and n >= 320 and not (d == 128 and wide and cap > 64 and Hv <= 2 ** 15) else 1)
        assert Hv <= 2 ** 15 or heads == (2 if grouped else 1)
