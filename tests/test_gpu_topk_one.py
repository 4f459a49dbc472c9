"""The block top-k of small selections in one workgroup per block: blocks that
the workgroup streams itself (up to 65536 elements) and blocks reduced by the
launch before it, candidates of one chunk (16384) and of several, ties that
straddle chunks, thresholds that collapse, keys further apart than the
fine bins reach, k_blk from 1 to the largest (4096) and one past it, lazy
receipts.  Bit for bit against the oracle."""

import numpy as np
import pytest
import torch

from oracle import spardl_oracle as so
from paper_2304_00737_amd import workloads as W
from tests.gpu_util import check_ws, compare_lazy_step, compare_step, log

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


# blocks of 1 element; 65536 and one more (ragged); one chunk and several of ties; tiles up to the 1024th
SIZES = [(3, 3, 1), (4, 4 * 65536, 4096), (4, 4 * 65536 + 4, 300), (2, 131_075, 4095), (3, 300_000, 1), (2, 250_000, 4096),
         (2, 250_000, 4097), (1, 2_097_000, 700), (1, 2_100_000, 700)]


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


# blocks of 16384 elements (all of them fit), 65536 (the workgroup streams them), 65537 and 2^18 (the launch before it)
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
