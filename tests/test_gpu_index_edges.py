"""GPU tests of the block-index build at the sizes where its passes change:
masks shorter than one wide load, rows and columns around the 16-byte and
64-entry pieces, runs too long for the LDS staging, more lists than the
in-fill sums take, and a capacity below the entry count. Bit-exact against
the oracle's lists (paper Sec. 3.3, Eq. 7)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_23169_amd as ut

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _mask(seed, shape, density):
    return (np.random.default_rng(seed).random(shape) < density).astype(np.uint8)


def _check(bm):
    got = ut.build_block_index(torch.from_numpy(bm).to(DEV))
    ref = oracle.block_index(bm)
    for key, want in zip(("q_rowptr", "q_cols", "kv_colptr", "kv_rows"), ref):
        have = got[key].cpu().numpy()[:len(want)]
        assert np.array_equal(have, want), key
    assert got["nnz"] == int(ref[0][-1])


@pytest.mark.parametrize("shape,density", [
    ((1, 1, 1, 1), 1.0), ((1, 1, 1, 3), 0.7), ((1, 1, 3, 5), 0.5),     # below 16 bytes
    ((1, 1, 2, 8), 0.5), ((1, 1, 17, 1), 0.5), ((1, 3, 4, 15), 0.4),    # 16 bytes and a little more
    ((2, 3, 63, 65), 0.3), ((1, 2, 64, 64), 1.0), ((1, 2, 65, 63), 0.3),
    ((1, 1, 70, 1023), 0.2), ((1, 1, 70, 1025), 0.2),                   # two loads per row
    ((1, 1, 1025, 70), 0.2), ((1, 1, 2111, 40), 0.3),                   # several tiles per wave
    ((1, 2, 600, 601), 1.0), ((1, 2, 448, 448), 1.0),                   # past and at the staged run
    ((1, 1, 601, 600), 0.75),
    ((1, 64, 256, 9), 0.3), ((1, 64, 257, 9), 0.3),                     # rows at and past the sums
    ((1, 64, 9, 257), 0.3),                                             # columns past them
    ((1, 5, 33, 77), 0.0),
    ((1, 24, 6, 6), 0.4), ((1, 1, 4, 4), 0.6), ((1, 1, 4, 5), 0.6),     # every slab reads past the end
    ((1, 1, 1, 1019), 0.9), ((1, 1, 2, 1021), 0.9),                     # 1 to 15 bytes of the last load
    ((1, 1, 3, 1030), 0.9), ((1, 1, 1, 31), 1.0),
])
def test_edges(shape, density):
    _check(_mask(sum(shape), shape, density))


def test_small_masks_take_no_longer_than_larger_ones():
    """All of a small mask's slabs read near its end, which is clamped and
    shifted there; byte by byte, 30 blocks took longer than 52."""
    def us(nb):
        bm = torch.from_numpy(_mask(nb, (1, 24, nb, nb), 0.3)).to(DEV)
        ut.build_block_index(bm)
        ut.ut_trace_enable(1)
        try:
            for _ in range(50):
                ut.build_block_index(bm)
            return sum(t["total_ms"] for t in ut.trace_read()) * 20
        finally:
            ut.ut_trace_enable(0)

    us(52)
    large = min(us(52) for _ in range(3))
    for nb in (6, 30):
        small = min(us(nb) for _ in range(3))
        assert small < 1.1 * large, (nb, small, large)


def test_capacity_below_the_entries():
    """Entries past the capacity are not written; the pointers are whole."""
    bm = _mask(5, (1, 2, 130, 130), 0.4)
    ref = oracle.block_index(bm)
    cap = int(ref[0][-1]) // 2
    rp, cp = (torch.zeros(2 * 130 + 1, dtype=torch.int32, device=DEV) for _ in range(2))
    cols, rows = (torch.full((cap + 64,), -7, dtype=torch.int32, device=DEV) for _ in range(2))
    st, nnz = ut.ut_build_block_index(torch.from_numpy(bm).to(DEV), rp, cols[:cap], cp, rows[:cap],
                                      nnz_host=True)
    assert st == ut.UT_ERR_CAPACITY and nnz == int(ref[0][-1])
    for got, want in ((rp, ref[0]), (cp, ref[2])):
        assert np.array_equal(got.cpu().numpy(), want)
    for got, want in ((cols, ref[1]), (rows, ref[3])):
        got = got.cpu().numpy()
        assert np.array_equal(got[:cap], want[:cap]) and (got[cap:] == -7).all()


def test_repeated_builds_agree():
    """The fill's sums may meet counts or offsets of other workgroups; the
    lists are the same every time."""
    bm = torch.from_numpy(_mask(9, (1, 24, 300, 300), 0.1)).to(DEV)
    first = ut.build_block_index(bm)
    for _ in range(20):
        again = ut.build_block_index(bm)
        for key in ("q_rowptr", "q_cols", "kv_colptr", "kv_rows"):
            assert torch.equal(first[key], again[key]), key
