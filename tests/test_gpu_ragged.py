"""Ragged rows and blocks through the float4 residual add: block bounds, row
strides and base addresses that are no multiples of a float4, rows shorter
than one, tiles that end one element past or short of a block; the fused
add's candidates and collection hold there too.  Bit for bit against the
oracle (every value has one IEEE sum, so there is no tolerance)."""

import numpy as np
import pytest
import torch

from oracle import spardl_oracle as so
from paper_2304_00737_amd import workloads as W
from tests.gpu_util import assert_bits_equal, check_ws, compare_step, log, ws_spec_ok

pytestmark = pytest.mark.gpu
spardl = pytest.importorskip("paper_2304_00737_amd.spardl")

# rows shorter than a float4, of one, of a few; blocks a tile (2048) long and one
# element more or less; 14 and 6 workers with lengths no block size divides
SIZES = [(1, 1, 1), (2, 3, 1), (3, 3, 1), (1, 4, 2), (2, 5, 1), (3, 7, 2), (2, 9, 4), (5, 67, 3),
         (2, 4094, 20), (2, 4097, 20), (3, 6145, 33), (3, 12287, 100), (6, 40001, 70), (14, 100003, 71)]


@pytest.mark.parametrize("collect", ["fused", "separate", "plain"])
@pytest.mark.parametrize("P,n,kb", SIZES)
def test_ragged_steps(P, n, kb, collect):
    log(f"ragged step P={P} n={n} kb={kb} {collect}")
    st = spardl.SparDLStep(P, n, kb, fused=collect != "plain", fuse_collect=collect == "fused")
    acc = np.zeros((P, n), np.float32)
    for t in range(4):
        grad = W.small_rows("normal" if t != 2 else "ties", P, n, 31 * t + n)
        st.step(torch.from_numpy(grad).cuda())
        check_ws(st)
        res = so.spardl_step([acc[w] for w in range(P)], [grad[w] for w in range(P)], P, n, kb)
        compare_step(st, res, P, n, kb, residual=collect != "fused")
    if collect == "fused" and n > 4096:
        st.step(torch.from_numpy(W.small_rows("normal", P, n, 7)).cuda())
        st.step(torch.from_numpy(W.small_rows("normal", P, n, 8)).cuda())
        assert all(ws_spec_ok(st)), "ragged blocks keep the speculative candidates"


@pytest.mark.parametrize("off_a,off_g,pad", [(0, 1, 0), (1, 0, 1), (2, 3, 2), (3, 3, 31), (0, 0, 3)])
@pytest.mark.parametrize("P,n", [(3, 5), (4, 8192), (5, 9001)])
def test_add_any_address(P, n, off_a, off_g, pad):
    """Rows at any 4-byte address and any stride, with and without the fused
    histogram: nothing outside the rows is written."""
    log(f"add any address P={P} n={n} acc+{off_a} grad+{off_g} ld=n+{pad}")
    ld = n + pad
    for ws in (None, spardl.workspace(P, P, n, 1)):
        a = np.random.default_rng(n + pad).standard_normal(P * ld + 8).astype(np.float32)
        g = np.random.default_rng(n + 1).standard_normal(P * ld + 8).astype(np.float32)
        at, gt = torch.from_numpy(a).cuda(), torch.from_numpy(g).cuda()
        spardl.residual_add(at.data_ptr() + 4 * off_a, gt.data_ptr() + 4 * off_g, P, n, P if ws is not None else 0,
                            ws, 1, ld_acc=ld, ld_grad=ld)
        want = a.copy()
        for w in range(P):
            s, q = off_a + w * ld, off_g + w * ld
            want[s:s + n] = so.residual_add(a[s:s + n], g[q:q + n])
        assert_bits_equal(at.cpu().numpy(), want, "rows and what surrounds them")


def test_plain_add_many_rows():
    """More rows than one launch's grid holds."""
    log("plain add of 70000 rows of 3")
    a, g = torch.randn(70000, 3, device="cuda"), torch.randn(70000, 3, device="cuda")
    want = a + g
    spardl.residual_add(a, g, 70000, 3)
    assert torch.equal(a, want)


@pytest.mark.parametrize("rows", [0, 1])
@pytest.mark.parametrize("n,kb", [(2 ** 26, 1000), (2 ** 26 - 1, 1000), (2 ** 26 + 3, 1000),
                                  (2 ** 26, 2 ** 19), (2 ** 26, 2 ** 19 + 1)])
def test_collection_in_the_add_or_before_it(n, kb, rows):
    """Both sides of the sizes and densities where the deferred collection
    moves between the add's tiles and kernels before it: the same steps as
    with the collection as its own call."""
    P = 2
    log(f"collection in the add or before it n={n} kb={kb} rows={rows}")
    deferred = spardl.SparDLStep(P, n, kb, rows_per_call=rows, fuse_collect=True)
    own = spardl.SparDLStep(P, n, kb, rows_per_call=rows)
    gen = torch.Generator(device="cuda").manual_seed(n + kb)
    grad = torch.empty((P, n), device="cuda")
    for t in range(3):
        grad.normal_(generator=gen)
        for st in (deferred, own):
            st.step(grad)
            check_ws(st)
        assert torch.equal(deferred.dense, own.dense), f"update of step {t + 1}"
        assert torch.equal(deferred.local_idx, own.local_idx), f"selections of step {t + 1}"
    deferred.flush()
    check_ws(deferred)
    assert torch.equal(deferred.acc.view(torch.int32), own.acc.view(torch.int32)), "residual"


# P, n, kb, rows per call: calls of 3 2^24 elements (of steps of at least 2^27) and one less, a last group of fewer
# rows in the tiles and the others not, one worker
@pytest.mark.parametrize("P,n,kb,rows", [(4, 3 * 2 ** 24, 1000, 1), (4, 3 * 2 ** 24 - 1, 1000, 1), (3, 3 * 2 ** 24 + 1, 1000, 2),
                                         (5, 2 ** 25, 1000, 2), (5, 2 ** 25, 2 ** 16, 3), (8, 2 ** 24, 1000, 2),
                                         (8, 2 ** 24, 1000, 3), (1, 2 ** 27, 9000, 0), (1, 2 ** 27 - 1, 9000, 0)])
def test_collection_in_the_add_or_before_it_by_rows(P, n, kb, rows):
    """The route of the deferred collection follows the rows of the call (its
    index is built for all of them): the same steps as with the collection as
    its own call."""
    log(f"collection in the add or before it P={P} n={n} kb={kb} rows={rows}")
    deferred = spardl.SparDLStep(P, n, kb, rows_per_call=rows, fuse_collect=True)
    own = spardl.SparDLStep(P, n, kb, rows_per_call=rows)
    gen = torch.Generator(device="cuda").manual_seed(n + kb)
    grad = torch.empty((P, n), device="cuda")
    for t in range(3):
        grad.normal_(generator=gen)
        for st in (deferred, own):
            st.step(grad)
            check_ws(st)
        assert torch.equal(deferred.dense, own.dense), f"update of step {t + 1}"
        assert torch.equal(deferred.local_idx, own.local_idx), f"selections of step {t + 1}"
    deferred.flush()
    check_ws(deferred)
    assert torch.equal(deferred.acc.view(torch.int32), own.acc.view(torch.int32)), "residual"


# the collection in the add's tiles; before the add, even and ragged rows
@pytest.mark.parametrize("n,kb", [(4096, 40), (2 ** 26, 1000), (2 ** 26 + 3, 1000)])
def test_unsorted_drops_are_reported(n, kb):
    """A drop list that is not sorted inside its block sets the error word when
    its index is built, wherever the collection will run."""
    P = 2
    log(f"unsorted drops n={n} kb={kb}")
    st = spardl.SparDLStep(P, n, kb, fuse_collect=True)
    gen = torch.Generator(device="cuda").manual_seed(n)
    st.step(torch.empty((P, n), device="cuda").normal_(generator=gen))
    check_ws(st)
    assert int(st.drop_cnt[0][0, 0]) >= 2
    st.drop_idx[0][0, 0, :2] = st.drop_idx[0][0, 0, :2].flip(0)
    spardl.residual_collect_index(0, P, n, P, kb, st.drop_idx, st.drop_cnt, st.ws)
    assert spardl.ws_error(st.ws) & 64, "ERR_DROPS"


# in the add's tiles; before the add: the top-k ended by one workgroup, by the general emit (a slot, 2 and 8 per wave)
@pytest.mark.parametrize("P,n,kb", [(2, 2 ** 22, 1000), (64, 2 ** 21 + 64, 30), (2, 2 ** 26, 5000), (2, 2 ** 26 + 3, 100_000),
                                    (4, 2 ** 28, 1_000_000), (2, 2 ** 29, 40_000)])
@pytest.mark.parametrize("rows", [0, 1])
def test_deferred_collection_does_not_read_local_idx(P, n, kb, rows):
    """A caller may reuse local_idx once a step is done: spoiled here between
    two steps, the residual is that of a collection as its own call."""
    log(f"local_idx spoiled before a deferred collection P={P} n={n} kb={kb} rows={rows}")
    deferred = spardl.SparDLStep(P, n, kb, rows_per_call=rows, fuse_collect=True)
    own = spardl.SparDLStep(P, n, kb, rows_per_call=rows)
    gen = torch.Generator(device="cuda").manual_seed(n + kb)
    grad = torch.empty((P, n), device="cuda")
    for t in range(3):
        grad.normal_(generator=gen)
        deferred.local_idx.fill_(-1)
        for st in (deferred, own):
            st.step(grad)
            check_ws(st)
        assert torch.equal(deferred.dense, own.dense), f"update of step {t + 1}"
    deferred.flush()
    assert torch.equal(deferred.acc.view(torch.int32), own.acc.view(torch.int32)), "residual"
