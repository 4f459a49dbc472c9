"""A block whose threshold fell below its histogram's floor is counted again
from acc: blocks of every remainder of a float4, shorter than one, and longer
than a workgroup's pass, for selections ended by one workgroup and by the
general path; one whose threshold rises by up to 15 binades is not.  Bit for bit
against the oracle."""

import numpy as np
import pytest
import torch

from oracle import spardl_oracle as so
from tests.gpu_util import assert_bits_equal, assert_idx_equal, log

pytestmark = pytest.mark.gpu
spardl = pytest.importorskip("paper_2304_00737_amd.spardl")


@pytest.mark.parametrize("P,n,kb", [(1, 1, 1), (1, 3, 2), (1, 4, 1), (1, 5, 4), (2, 16_387, 40), (3, 49_151, 16),
                                    (1, 65_539, 300), (2, 131_077, 4097), (3, 200_003, 5000)])
def test_threshold_falls(P, n, kb):
    log(f"threshold falls P={P} n={n} kb={kb}")
    bounds = so.block_bounds(n, P)
    ws = spardl.workspace(P, P, n, kb)
    acc = torch.zeros((P, n), device="cuda")
    sp_idx = torch.empty((P, P, kb), dtype=torch.int32, device="cuda")
    sp_val, local = torch.empty((P, P, kb), device="cuda"), torch.empty_like(sp_idx)
    rng = np.random.default_rng(n)
    for scale in (1.0, 1e-4, 3.0, 1e-30, 0.0):
        g = (rng.standard_normal((P, n)) * scale).astype(np.float32) + np.float32(0.0)   # (acc + grad has no -0)
        acc.zero_()
        spardl.residual_add(acc, torch.from_numpy(g).cuda(), P, n, P, ws, kb)
        spardl.block_topk(acc, P, n, P, kb, sp_idx, sp_val, local, ws, spardl.TOPK_HIST_READY)
        assert spardl.ws_error(ws) == 0
        for w in range(P):
            for b in range(P):
                want_i, want_v = so.local_sparsify(g[w, bounds[b]:bounds[b + 1]], bounds[b], kb)
                assert_idx_equal(sp_idx[w, b].cpu().numpy(), want_i, f"indices w={w} b={b} scale={scale}")
                assert_bits_equal(sp_val[w, b].cpu().numpy(), want_v, f"values w={w} b={b} scale={scale}")


@pytest.mark.parametrize("P,n,kb", [(2, 200_000, 300), (2, 200_000, 5000), (3, 400_003, 4097)])
@pytest.mark.parametrize("binades", [6, 7, 8, 9, 12, 15])
def test_threshold_rises(P, n, kb, binades):
    """Up to 15 binades above the step before, the histogram still tells the
    threshold bin: acc, spoiled here after the add, is not read again."""
    log(f"threshold rises P={P} n={n} kb={kb} by 2^{binades}")
    bounds = so.block_bounds(n, P)
    ws = spardl.workspace(P, P, n, kb)
    acc = torch.zeros((P, n), device="cuda")
    sp_idx = torch.empty((P, P, kb), dtype=torch.int32, device="cuda")
    sp_val, local = torch.empty((P, P, kb), device="cuda"), torch.empty_like(sp_idx)
    g = np.random.default_rng(n + binades).standard_normal((P, n)).astype(np.float32)
    for scale in (1.0, 2.0 ** binades):
        acc.zero_()
        spardl.residual_add(acc, torch.from_numpy(g * np.float32(scale)).cuda(), P, n, P, ws, kb)
        if scale != 1.0:
            acc.fill_(float("inf"))
        spardl.block_topk(acc, P, n, P, kb, sp_idx, sp_val, local, ws, spardl.TOPK_HIST_READY)
        assert spardl.ws_error(ws) == 0
    for w in range(P):
        for b in range(P):
            want_i, want_v = so.local_sparsify(g[w, bounds[b]:bounds[b + 1]] * np.float32(scale), bounds[b], kb)
            assert_idx_equal(sp_idx[w, b].cpu().numpy(), want_i, f"indices w={w} b={b}")
            assert_bits_equal(sp_val[w, b].cpu().numpy(), want_v, f"values w={w} b={b}")
