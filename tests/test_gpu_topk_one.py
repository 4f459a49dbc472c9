"""The block top-k of small selections, ended by one workgroup per block: blocks
that the workgroup streams itself (up to 65536 elements) and blocks filtered
by the launches before it, candidates of one chunk (16384) and of several, ties
and zeros that straddle chunks and slots, thresholds that collapse, keys further
apart than the fine bins reach, k_blk from 1 to the largest (4096) and one past
it, lists taken as the add left them, lazy receipts.  Bit for bit against the
oracle."""

import numpy as np
import pytest
import torch

from oracle import spardl_oracle as so
from paper_2304_00737_amd import workloads as W
from tests.gpu_util import assert_bits_equal, assert_idx_equal, check_ws, compare_lazy_step, compare_step, log

pytestmark = pytest.mark.gpu
spardl = pytest.importorskip("paper_2304_00737_amd.spardl")


def _grad(P, n, t):
    """Step t's gradients: normal, with a few huge entries (far above the fine
    bins), all ties (every entry a candidate), tiny ones after large (a collapse
    once the large ones are sent), wide (eight decades)."""
    rng = np.random.default_rng(17 * t + n)
    g = W.small_rows("normal", P, n, 4000 + 10 * t + P)
    if t == 1:
        g[:, rng.choice(n, max(1, n // 1000), replace=False)] *= np.float32(1e12)
    if t == 2:
        g = W.small_rows("const", P, n, 0)
    if t == 3:
        g *= np.float32(1e-6)
    if t == 4:
        g *= np.float32(10.0) ** rng.integers(-4, 5, size=(P, n)).astype(np.float32)
    return g


# blocks of 1 element; 65536 and one more (ragged); one chunk and several of ties; tiles up to the 1024th; calls
# with 3825 slots and, from 4096 on, with 4352 (the add's lists are taken as they are)
SIZES = [(3, 3, 1), (4, 4 * 65536, 4096), (4, 4 * 65536 + 4, 300), (2, 131_075, 4095), (3, 300_000, 1), (2, 250_000, 4096),
         (2, 250_000, 4097), (1, 2_097_000, 700), (1, 2_100_000, 700), (15, 15 * 65_600, 30), (16, 16 * 65_600 + 5, 30)]


@pytest.mark.parametrize("collect", ["fused", "plain"])
@pytest.mark.parametrize("P,n,kb", SIZES)
def test_topk_one_steps(P, n, kb, collect):
    st = spardl.SparDLStep(P, n, kb, fused=collect != "plain", fuse_collect=collect == "fused")
    acc = np.zeros((P, n), np.float32)
    for t in range(6):
        log(f"topk in one workgroup P={P} n={n} kb={kb} {collect} step {t + 1}")
        grad = _grad(P, n, t)
        st.step(torch.from_numpy(grad).cuda())
        check_ws(st)
        res = so.spardl_step([acc[w] for w in range(P)], [grad[w] for w in range(P)], P, n, kb)
        compare_step(st, res, P, n, kb, residual=collect != "fused")


@pytest.mark.parametrize("P,n,kb", [(4, 200_000, 300), (3, 250_001, 4096)])
def test_topk_one_lazy(P, n, kb):
    st = spardl.SparDLLazyStep(P, n, kb)
    acc = np.zeros((P, n), np.float32)
    for t in range(5):
        log(f"lazy topk in one workgroup P={P} n={n} kb={kb} step {t + 1}")
        grad = _grad(P, n, t)
        st.step(torch.from_numpy(grad).cuda())
        check_ws(st)
        res = so.spardl_step_lazy([acc[w] for w in range(P)], [grad[w] for w in range(P)], P, n, kb)
        compare_lazy_step(st, res, P, n, kb)


# blocks of 16384 elements (all of them fit), 65536 (the workgroup streams them), 65537 and 2^18 (the launches before it)
@pytest.mark.parametrize("P,n,kb", [(4, 4 * 16384, 300), (4, 4 * 65536, 4096), (2, 2 * 65537, 300), (4, 1 << 20, 2622)])
def test_topk_one_piled_up(P, n, kb):
    """A residual piled up just below the threshold: a third, then all of a
    block within the candidates' margin, on both sides of what the registers hold."""
    st = spardl.SparDLStep(P, n, kb, fuse_collect=True)
    acc = np.zeros((P, n), np.float32)
    rng = np.random.default_rng(n)
    for t in range(6):
        log(f"topk in one workgroup, piled up P={P} n={n} kb={kb} step {t + 1}")
        grad = np.float32(1e-3) * rng.standard_normal((P, n)).astype(np.float32)
        if t in (0, 3):
            some = rng.random((P, n)) < (0.33 if t == 0 else 1.0)
            grad[some] = (rng.choice([-1.0, 1.0], n * P) * rng.uniform(1.0, 1.05, n * P)).astype(np.float32).reshape(P, n)[some]
        st.step(torch.from_numpy(grad).cuda())
        check_ws(st)
        res = so.spardl_step([acc[w] for w in range(P)], [grad[w] for w in range(P)], P, n, kb)
        compare_step(st, res, P, n, kb, residual=False)


# one slot and a bit more than the registers hold; a block's last slot of one element; the longest; ragged bounds
@pytest.mark.parametrize("P,n,kb", [(4, 4 * 16384, 700), (2, 2 * 65536, 4096), (2, 131_073, 4096), (1, 69 * 4096 + 1, 33),
                                    (3, 700_001, 4096), (1, 2_097_000, 4096)])
def test_topk_one_mostly_zeros(P, n, kb):
    """Blocks with fewer non-zero entries than they select, whose threshold is
    zero step after step, so every entry is a candidate: few non-zeros, none at
    all, and as many as are selected; signed zeros tie."""
    st = spardl.SparDLStep(P, n, kb)
    acc = np.zeros((P, n), np.float32)
    rng = np.random.default_rng(n)
    for t, nz in enumerate([kb // 4, 0, kb, kb // 2]):
        log(f"topk in one workgroup, mostly zeros P={P} n={n} kb={kb} step {t + 1}")
        grad = np.where(rng.random((P, n)) < 0.5, np.float32(0.0), np.float32(-0.0)).astype(np.float32)
        for w in range(P):
            grad[w, rng.choice(n, nz, replace=False)] = rng.standard_normal(nz).astype(np.float32)
        st.step(torch.from_numpy(grad).cuda())
        check_ws(st)
        res = so.spardl_step([acc[w] for w in range(P)], [grad[w] for w in range(P)], P, n, kb)
        compare_step(st, res, P, n, kb)


# one past the registers' 16384; many; ragged blocks
@pytest.mark.parametrize("P,n,kb,cands", [(2, 1 << 19, 700, 16385), (1, 2_000_000, 1000, 20_000), (2, 1_999_999, 4096, 300_000),
                                          (16, 16 * 65_600, 30, 100)])
def test_topk_one_takes_the_adds_candidates(P, n, kb, cands):
    """The candidates the add left decide a block however many they are: the
    values in acc are not read again (they are spoiled here after the add)."""
    log(f"the add's candidates P={P} n={n} kb={kb} candidates per block {cands}")
    bounds = so.block_bounds(n, P)
    rng = np.random.default_rng(n)
    ws = spardl.workspace(P, P, n, kb)
    acc = torch.zeros((P, n), device="cuda")
    sp_idx = torch.empty((P, P, kb), dtype=torch.int32, device="cuda")
    sp_val, local = torch.empty((P, P, kb), device="cuda"), torch.empty_like(sp_idx)
    for t in range(2):
        g = np.float32(1e-3) * rng.standard_normal((P, n)).astype(np.float32)
        for w in range(P):
            for s, e in zip(bounds[:-1], bounds[1:]):   # within the two bins below the threshold that the add keeps
                g[w, s + rng.choice(e - s, cands, replace=False)] = rng.uniform(1.0, 1.03, cands).astype(np.float32)
        acc.zero_()
        spardl.residual_add(acc, torch.from_numpy(g).cuda(), P, n, P, ws, kb)
        if t == 1:
            acc.fill_(float("inf"))
        spardl.block_topk(acc, P, n, P, kb, sp_idx, sp_val, local, ws, spardl.TOPK_HIST_READY)
        assert spardl.ws_error(ws) == 0
    for w in range(P):
        for b in range(P):
            want_i, want_v = so.local_sparsify(g[w, bounds[b]:bounds[b + 1]], bounds[b], kb)
            assert_idx_equal(sp_idx[w, b].cpu().numpy(), want_i, f"indices w={w} b={b}")
            assert_bits_equal(sp_val[w, b].cpu().numpy(), want_v, f"values w={w} b={b}")


# blocks the workgroup has alone, blocks filtered before it, blocks whose lists it takes as they are, the general path
@pytest.mark.parametrize("P,n,kb", [(4, 4 * 4096, 41), (2, 2 * 65_536, 300), (2, 1 << 19, 700), (16, 16 * 65_600, 30),
                                    (2, 200_000, 5000)])
@pytest.mark.parametrize("before", [0, 1, 2])
def test_two_adds_before_a_topk(P, n, kb, before):
    """A second add before the block top-k leaves histograms of twice the
    entries: the error word says so, in a block's first step and in later ones,
    and a prepared workspace works again."""
    log(f"two adds before a top-k P={P} n={n} kb={kb} after {before} steps")
    ws = spardl.workspace(P, P, n, kb)
    acc = torch.zeros((P, n), device="cuda")
    sp_idx = torch.empty((P, P, kb), dtype=torch.int32, device="cuda")
    sp_val, local = torch.empty((P, P, kb), device="cuda"), torch.empty_like(sp_idx)
    gen = torch.Generator(device="cuda").manual_seed(n)

    def step(adds):
        for _ in range(adds):
            spardl.residual_add(acc, torch.empty_like(acc).normal_(generator=gen), P, n, P, ws, kb)
        spardl.block_topk(acc, P, n, P, kb, sp_idx, sp_val, local, ws, spardl.TOPK_HIST_READY)
        return spardl.ws_error(ws)

    for _ in range(before):
        assert step(1) == 0
    assert step(2) & 2, "the histograms hold more than the blocks"
    spardl.workspace_init(ws, P, P, n, kb)
    for _ in range(2):
        assert step(1) == 0
