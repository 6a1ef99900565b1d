"""How mdlg_displacement_hist deals its work to blocks: the rule (csrc/hist_shares.h,
host arithmetic) compiled on its own.  A block counts in 32 bits, 512 particles an
axis and item, so no block may take 2^32 / 512 items or more, however many blocks the
launch has."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """#include "hist_shares.h"
extern "C" void deal(int n_rep, const long long* items, int n_lag, long long* shares) {
    mdlg::hist_deal(n_rep, items, n_lag, shares);
}
extern "C" int item(void) { return mdlg::kHistItem; }
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("hist_shares")
    (d / "deal.cpp").write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2101_01160_amd", "csrc"), str(d / "deal.cpp"), "-o", str(d / "deal.so")],
                   check=True)
    lib = C.CDLL(str(d / "deal.so"))

    def deal(items, n_lag):
        a = np.asarray(items, dtype=np.int64)
        out = np.full(len(a), -7, dtype=np.int64)
        lib.deal(C.c_int(len(a)), a.ctypes.data_as(C.c_void_p), C.c_int(n_lag), out.ctypes.data_as(C.c_void_p))
        return out

    deal.item = lib.item()
    return deal


@pytest.mark.parametrize("n_rep,n_lag", [(1, 1), (5, 64), (32, 16), (32, 64), (4, 64), (5, 52)])
@pytest.mark.parametrize("most", [1, 2, 511, 2**22 - 1, 2**22, 2**22 + 1, 2**23 - 1, 2**23, 2**24 - 1, 2**24, 2**30 + 3])
def test_no_block_counts_to_2_32(rule, n_rep, n_lag, most):
    items = [most] + [max(1, most // 1000)] * (n_rep - 1)
    shares = rule(items, n_lag)
    for n, k in zip(items, shares):
        assert k >= 1
        # block b of k takes the items from n b / k up to n (b + 1) / k
        worst = -(-n // int(k)) * rule.item
        assert worst < 2**32


def test_replicas_without_particles(rule):
    assert (rule([0, 7, 0], 2) >= 0).all()


@pytest.mark.parametrize("items,n_lag", [([18000] + [64] * 31, 1), ([64] * 31 + [18000], 16), ([18000, 0, 0, 1], 4),
                                         ([5, 3], 64), ([2**23 - 1] + [8] * 255, 1)])
def test_blocks_follow_the_work(rule, items, n_lag):
    """The launch has about 512 blocks, and no replica is left with much more work per block than all have together;
    one without work has none."""
    shares = rule(items, n_lag)
    target = max(1, 512 // n_lag)
    assert shares.sum() <= target + len(items)
    for n, k in zip(items, shares):
        assert (k == 0) == (n == 0)
        if k:
            # floor(target n / total) + 1 > target n / total, so the items of a block stay below twice the average
            assert -(-n // int(k)) <= max(2 * sum(items) // target, 1) + 1
