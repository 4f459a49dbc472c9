"""Bit-exact parity of the HIP path (through the C ABI) with the CPU oracle.

Tolerance is zero everywhere: indices must be equal and fp32 values must have
identical bit patterns.  Sizes span several tiles of every kernel plus ragged
tails; edge cases cover P = 1, k/P = 1, k/P = block length, giant ties, all
zeros, signed zeros, subnormals and n not divisible by P or by 4.
"""

import numpy as np
import pytest

from oracle import spardl_oracle as so
from tests.conftest import gpu_available
from tests.gpu_util import assert_bits_equal, assert_idx_equal, check_ws, compare_step, log, ws_spec_ok

pytestmark = pytest.mark.gpu

if gpu_available():
    import torch
    from paper_2304_00737_amd import spardl
    from paper_2304_00737_amd import workloads as W


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _rows(kind, P, n, seed):
    return W.small_rows(kind, P, n, seed)


# --------------------------------------------------------------------------- a1


@pytest.mark.parametrize("P,n,ld,hist", [(4, 1 << 20, 1 << 20, True), (3, 1001, 1001, True),
                                         (2, 4099, 4200, False), (5, 40000, 40000, False),
                                         (8, 8000, 8000, True)])
def test_residual_add(P, n, ld, hist):
    log(f"residual_add P={P} n={n} ld={ld} hist={hist}")
    rng = np.random.default_rng(n)
    acc = np.zeros((P, ld), np.float32)
    grad = np.zeros((P, ld), np.float32)
    acc[:, :n] = rng.standard_normal((P, n)).astype(np.float32)
    grad[:, :n] = rng.standard_normal((P, n)).astype(np.float32)
    # specials: subnormals, signed zeros, exact cancellation, large magnitudes
    sub = np.array([1e-45, -1e-45, 1e-40, -3e-39], np.float32)
    acc[0, :4] = sub
    grad[0, :4] = sub[::-1]
    acc[0, 4:8] = [0.0, -0.0, 1.5, 3e38]
    grad[0, 4:8] = [-0.0, -0.0, -1.5, 3e38]
    a_d, g_d = _dev(acc), _dev(grad)
    ws = None
    if hist:
        ws = spardl.workspace(P, P, n, 1)
    spardl.residual_add(a_d, g_d, P, n, P if hist else 0, ws, 1 if hist else 0, ld_acc=ld, ld_grad=ld)
    want = acc.copy()
    want[:, :n] = so.residual_add(acc[:, :n], grad[:, :n])
    assert_bits_equal(a_d.cpu().numpy(), want, "acc after residual add")


# --------------------------------------------------------------------------- a3

TOPK_CASES = [
    (4, 1 << 20, 2622, "normal"),
    (1, 5000, 7, "normal"),
    (2, 10007, 3, "ties"),
    (3, 6000, 1, "ties"),
    (5, 6000, 1200, "normal"),
    (7, 10007, 3, "const"),
    (6, 6000, 5, "zeros"),
    (14, 10007, 3, "ties"),
    (12, 6000, 1, "dyadic"),
    (8, 300000, 400, "ties"),
    (16, 1 << 18, 100, "normal"),
    (3, 100003, 33334, "dyadic"),
    (2, 200000, 1000, "const"),        # a 100000-entry threshold bin: several register chunks
    (4, 400000, 5000, "ties"),
]


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("P,n,kb,kind", TOPK_CASES)
def test_block_topk(P, n, kb, kind, fused):
    log(f"block_topk P={P} n={n} kb={kb} kind={kind} fused={fused}")
    acc0 = _rows(kind, P, n, 1 + P)
    grad = _rows(kind, P, n, 2 + P)
    st = spardl.SparDLStep(P, n, kb, fused=fused)
    st.acc.copy_(_dev(acc0))
    st.residual_add(_dev(grad))
    st.block_topk()
    check_ws(st)
    A = so.residual_add(acc0, grad)
    bounds = so.block_bounds(n, P)
    sp_idx, sp_val = st.sp_idx.cpu().numpy(), st.sp_val.cpu().numpy()
    local = st.local_idx.cpu().numpy()
    for w in range(P):
        for b in range(P):
            oi, ov = so.local_sparsify(A[w, bounds[b]:bounds[b + 1]], bounds[b], kb)
            assert_idx_equal(sp_idx[w, b], oi, f"idx w={w} b={b}")
            assert_idx_equal(local[w, b], oi, f"local w={w} b={b}")
            assert_bits_equal(sp_val[w, b], ov, f"val w={w} b={b}")


def test_block_topk_subset_rows():
    """nworkers < P: one row at a time, as for very large gradients."""
    P, n, kb = 6, 60000, 77
    acc = _rows("ties", P, n, 5)
    a_d = _dev(acc)
    ws = spardl.workspace(1, P, n, kb)
    sp_i = torch.empty((P, P, kb), dtype=torch.int32, device="cuda")
    sp_v = torch.empty((P, P, kb), dtype=torch.float32, device="cuda")
    for w in range(P):
        spardl.block_topk(a_d[w], 1, n, P, kb, sp_i[w], sp_v[w], None, ws)
    assert spardl.ws_error(ws) == 0
    bounds = so.block_bounds(n, P)
    si, sv = sp_i.cpu().numpy(), sp_v.cpu().numpy()
    for w in range(P):
        for b in range(P):
            oi, ov = so.local_sparsify(acc[w, bounds[b]:bounds[b + 1]], bounds[b], kb)
            assert_idx_equal(si[w, b], oi, f"idx w={w} b={b}")
            assert_bits_equal(sv[w, b], ov, f"val w={w} b={b}")


# --------------------------------------------------------------------------- a4


def _random_state(P, n, kb, overlap, kind, seed):
    rng = np.random.default_rng(seed)
    bounds = so.block_bounds(n, P)
    idx = np.zeros((P, P, kb), np.int32)
    for w in range(P):
        for b in range(P):
            L = bounds[b + 1] - bounds[b]
            pool = L if overlap == "low" else min(L, kb + max(1, kb // 5))
            pool = kb if overlap == "full" else pool
            idx[w, b] = np.sort(rng.choice(pool, size=kb, replace=False)) + bounds[b]
    if kind == "outlier":
        # one entry per block 2^40 times the rest: the union's threshold lies
        # far below its largest key (a single-workgroup merge's level 1 then
        # takes the 1/16-binade bins)
        val = W.small_rows("normal", P * P, kb, seed + 1).reshape(P, P, kb)
        val[:, :, kb // 2] *= np.float32(2.0 ** 40)
    else:
        val = W.small_rows(kind, P * P, kb, seed + 1).reshape(P, P, kb)
    return idx, val


@pytest.mark.parametrize("P,kb,overlap,kind", [
    (2, 1, "full", "normal"), (3, 3, "high", "ties"), (5, 700, "high", "normal"),
    (6, 5000, "low", "normal"), (8, 2100, "high", "ties"), (14, 33, "full", "dyadic"),
    (4, 9000, "full", "ties"), (7, 4097, "high", "normal"), (16, 200, "low", "ties"),
    (4, 4096, "full", "normal"), (6, 300, "high", "outlier"), (5, 2000, "low", "zeros"),
])
def test_merge_rounds(P, kb, overlap, kind):
    log(f"merge P={P} kb={kb} overlap={overlap} kind={kind}")
    n = P * max(3 * kb, 64) + (P - 1)
    idx, val = _random_state(P, n, kb, overlap, kind, 1000 + P + kb)
    sp_i, sp_v = _dev(idx), _dev(val)
    l, dist, bags = spardl.srs_plan(P)
    ws = spardl.workspace(P, P, n, kb)
    sched = so.srs_schedule(P)
    assert [s.distance for s in sched] == dist
    for step in sched:
        m = bags[step.i - 1]
        pre_i, pre_v = sp_i.cpu().numpy(), sp_v.cpu().numpy()
        di = torch.full((P, m, kb), -7, dtype=torch.int32, device="cuda")
        dv = torch.zeros((P, m, kb), dtype=torch.float32, device="cuda")
        dc = torch.full((P, m), -1, dtype=torch.int32, device="cuda")
        spardl.sparse_merge_topk(sp_i, sp_v, P, n, kb, step.i, di, dv, dc, ws)
        assert spardl.ws_error(ws) == 0
        post_i, post_v = sp_i.cpu().numpy(), sp_v.cpu().numpy()
        di, dv, dc = di.cpu().numpy(), dv.cpu().numpy(), dc.cpu().numpy()
        touched = set()
        for w in range(P):
            src = step.source[w]
            assert [(w + t) % P for t in range(m)] == list(step.received_bag[w])
            for t, b in enumerate(step.received_bag[w]):
                ki, kv, oi, ov = so.merge_and_resparsify(pre_i[w, b], pre_v[w, b], pre_i[src, b], pre_v[src, b], kb)
                assert_idx_equal(post_i[w, b], ki, f"step {step.i} kept idx w={w} b={b}")
                assert_bits_equal(post_v[w, b], kv, f"step {step.i} kept val w={w} b={b}")
                assert dc[w, t] == len(oi), f"step {step.i} drop count w={w} b={b}"
                assert_idx_equal(di[w, t, :len(oi)], oi, f"step {step.i} drop idx w={w} b={b}")
                assert_bits_equal(dv[w, t, :len(oi)], ov, f"step {step.i} drop val w={w} b={b}")
                touched.add((w, b))
        for w in range(P):
            for b in range(P):
                if (w, b) not in touched:
                    assert_idx_equal(post_i[w, b], pre_i[w, b], "untouched block changed")
                    assert_bits_equal(post_v[w, b], pre_v[w, b], "untouched block changed")


# --------------------------------------------------------------------------- whole step


STEP_CASES = [
    (1, 4000, 9, "normal", 2),
    (2, 5000, 50, "ties", 2),
    (3, 6001, 1, "ties", 2),
    (4, 8192, 2048, "dyadic", 1),
    (5, 10007, 3, "normal", 2),
    (6, 6000, 1000, "ties", 2),
    (7, 70001, 501, "normal", 3),
    (8, 200000, 250, "ties", 2),
    (12, 60000, 50, "dyadic", 2),
    (14, 10007, 7, "const", 2),
    (16, 65536, 41, "normal", 2),
    (9, 9000, 1, "zeros", 1),
]


@pytest.mark.parametrize("P,n,kb,kind,steps", STEP_CASES)
def test_step(P, n, kb, kind, steps):
    log(f"step P={P} n={n} kb={kb} kind={kind} steps={steps}")
    st = spardl.SparDLStep(P, n, kb)
    acc = np.zeros((P, n), np.float32)
    for t in range(steps):
        grad = _rows(kind, P, n, 100 * t + P)
        st.step(_dev(grad))
        check_ws(st)
        res = so.spardl_step([acc[w] for w in range(P)], [grad[w] for w in range(P)], P, n, kb)
        compare_step(st, res, P, n, kb)


@pytest.mark.parametrize("P,n,kb,kind,steps", [STEP_CASES[i] for i in (1, 4, 6, 8)])
def test_step_unfused(P, n, kb, kind, steps):
    """Residual add without histogram, block top-k that counts the block
    itself and residual collection that builds I in the workspace."""
    log(f"step unfused P={P} n={n} kb={kb} kind={kind} steps={steps}")
    st = spardl.SparDLStep(P, n, kb, fused=False)
    acc = np.zeros((P, n), np.float32)
    for t in range(steps):
        grad = _rows(kind, P, n, 100 * t + P + 1)
        st.step(_dev(grad))
        check_ws(st)
        res = so.spardl_step([acc[w] for w in range(P)], [grad[w] for w in range(P)], P, n, kb)
        compare_step(st, res, P, n, kb)


FUSED_COLLECT_CASES = [STEP_CASES[i] for i in (0, 1, 2, 3, 4, 5, 6, 7, 8, 10)]


@pytest.mark.parametrize("rows", [0, 1, 3])
@pytest.mark.parametrize("P,n,kb,kind,steps", FUSED_COLLECT_CASES)
def test_step_fused_collect(P, n, kb, kind, steps, rows):
    """The residual collection left to the next step's add: after every add,
    acc equals the oracle's residual plus the gradient, bit for bit; every
    step's selections, drops and update are the oracle's; flush() leaves the
    last residual.  rows: workers per call (0: all).  At these sizes the
    collection runs in the add's tiles (large sparse steps, collected by
    kernels before it, are held against a collection of its own in
    test_gpu_ragged.py and against full-size checksums)."""
    if rows > P:
        pytest.skip("fewer workers than rows per call")
    log(f"step fused collect P={P} n={n} kb={kb} kind={kind} steps={steps + 1} rows={rows}")
    st = spardl.SparDLStep(P, n, kb, fuse_collect=True, rows_per_call=rows)
    acc = np.zeros((P, n), np.float32)
    for t in range(steps + 1):
        grad = _rows(kind, P, n, 100 * t + P + 7)
        g = _dev(grad)
        for w0 in range(0, P, st.rows):
            r = min(st.rows, P - w0)
            st.residual_add_rows(w0, g[w0:w0 + r])
            got = st.acc[w0:w0 + r].cpu().numpy()
            for w in range(w0, w0 + r):
                assert_bits_equal(got[w - w0], so.residual_add(acc[w], grad[w]), f"add step {t} worker {w}")
            st.block_topk_rows(w0, r)
        st.finish()
        check_ws(st)
        res = so.spardl_step([acc[w] for w in range(P)], [grad[w] for w in range(P)], P, n, kb)
        compare_step(st, res, P, n, kb, residual=False)
    st.flush()
    check_ws(st)
    for w in range(P):
        assert_bits_equal(st.acc[w].cpu().numpy(), acc[w], f"residual after flush worker {w}")


@pytest.mark.parametrize("P,n,kb,rows", [(8, 50000, 100, 1), (7, 70001, 501, 3), (5, 10007, 3, 2)])
def test_step_rows_per_call(P, n, kb, rows):
    """Workers a few at a time (a workspace for `rows` rows): the same step."""
    log(f"step rows_per_call={rows} P={P} n={n} kb={kb}")
    st = spardl.SparDLStep(P, n, kb, rows_per_call=rows)
    acc = np.zeros((P, n), np.float32)
    for t in range(3):
        grad = _rows("normal", P, n, 300 * t + P)
        st.step(_dev(grad))
        check_ws(st)
        res = so.spardl_step([acc[w] for w in range(P)], [grad[w] for w in range(P)], P, n, kb)
        compare_step(st, res, P, n, kb)


def test_threshold_hints_are_per_worker():
    """Workers taken one at a time on a one-row workspace: the previous
    threshold each fused add starts from is that worker's own, so after a
    step the hint of (worker w, block b) is the level-1 bin of the k/P-th
    largest |A| of worker w's block b (plus one), for every worker."""
    from paper_2304_00737_amd.spardl import ws_layout
    P, n, kb = 6, 60000, 40
    st = spardl.SparDLStep(P, n, kb, rows_per_call=1)
    acc = np.zeros((P, n), np.float32)
    L = ws_layout(P, n, kb, st.ws.numel())
    for t in range(3):
        # worker w's gradient scaled by 4^w: every worker's thresholds sit in different bins
        grad = (_rows("normal", P, n, 610 + t) * (np.float32(4.0) ** np.arange(P, dtype=np.float32))[:, None])
        grad = grad.astype(np.float32)
        st.step(_dev(grad))
        check_ws(st)
        res = so.spardl_step([acc[w] for w in range(P)], [grad[w] for w in range(P)], P, n, kb)
        compare_step(st, res, P, n, kb)
        hint = st.ws[L["spec_t1"]:L["spec_t1"] + P * P * 4].view(torch.int32).cpu().numpy()
        for w in range(P):
            for b in range(P):
                keys = np.asarray(res.local[(w, b)][1], np.float32).view(np.uint32) & 0x7FFFFFFF
                assert int(hint[w * P + b]) == int(keys.min() >> 19) + 1, f"hint of worker {w} block {b}"


def test_cfg1_full():
    wl = W.config(1)
    P, n, kb = wl.P, wl.n, wl.k_blk
    log(f"cfg1 {wl.describe()}")
    st = spardl.SparDLStep(P, n, kb)
    acc = np.zeros((P, n), np.float32)
    for t in range(1, wl.steps + 1):
        grad = np.stack([W.gradient(wl, t, w) for w in range(P)])
        st.step(_dev(grad))
        check_ws(st)
        res = so.spardl_step([acc[w] for w in range(P)], [grad[w] for w in range(P)], P, n, kb)
        compare_step(st, res, P, n, kb)


def test_deterministic():
    wl = W.config(1)
    P, n, kb = wl.P, wl.n, wl.k_blk
    grad = _dev(np.stack([W.gradient(wl, 1, w) for w in range(P)]))
    outs = []
    for rep in range(2):
        st = spardl.SparDLStep(P, n, kb)
        st.step(grad)
        st.step(grad)
        tensors = [st.acc, st.dense, st.sp_idx, st.sp_val, st.local_idx] + st.drop_cnt
        snap = [t.cpu().numpy().tobytes() for t in tensors]
        for di, dv, dc in zip(st.drop_idx, st.drop_val, st.drop_cnt):
            di, dv, dc = di.cpu().numpy(), dv.cpu().numpy(), dc.cpu().numpy()
            for w in range(P):
                for t in range(dc.shape[1]):     # only the valid prefix of each drop list
                    snap.append(di[w, t, :dc[w, t]].tobytes() + dv[w, t, :dc[w, t]].tobytes())
        outs.append(snap)
    assert outs[0] == outs[1]


def test_step_speculation_fallback():
    """The fused residual add writes candidates above a floor just below each
    block's previous threshold.  A much smaller gradient after a large one
    drops the threshold below that floor, so the top-k must read the block
    again; rising thresholds use the fused candidates.  Both paths must match
    the oracle bit for bit, and both must actually run."""
    P, n, kb = 4, 200000, 300
    st = spardl.SparDLStep(P, n, kb)
    acc = np.zeros((P, n), np.float32)
    bounds = so.block_bounds(n, P)
    rng = np.random.default_rng(77)
    used = []
    for t, scale in enumerate([1.0, 1e-4, 1.0, 1.0]):
        grad = (_rows("normal", P, n, 500 + t) * np.float32(scale)).astype(np.float32)
        if t == 0:   # k_blk huge entries per block: the top-k takes them, and the next threshold is far lower
            for w in range(P):
                for b in range(P):
                    pos = bounds[b] + rng.choice(bounds[b + 1] - bounds[b], kb, replace=False)
                    grad[w, pos] = np.float32(1000.0) * np.sign(grad[w, pos] + np.float32(0.5))
        log(f"speculation step {t + 1}: gradient scale {scale}")
        st.step(_dev(grad))
        check_ws(st)
        used.append(ws_spec_ok(st))
        res = so.spardl_step([acc[w] for w in range(P)], [grad[w] for w in range(P)], P, n, kb)
        compare_step(st, res, P, n, kb)
    assert not any(used[0]), "no speculation is possible on the first step"
    assert not all(used[1]), "a falling threshold must fall back to re-reading the block"
    assert all(used[3]), "rising thresholds use the fused candidates"


def test_histogram_misuse_is_flagged():
    """Two residual adds into one workspace without the top-k that consumes
    the histogram double-count it; the next top-k must flag the inconsistent
    total in the (sticky) error word, and workspace_init must clear it."""
    P, n, kb = 4, 40000, 50
    st = spardl.SparDLStep(P, n, kb)
    grad = _dev(_rows("normal", P, n, 77))
    st.residual_add(grad)
    st.residual_add(grad)
    st.block_topk()
    assert spardl.ws_error(st.ws) & spardl.WS_ERR_COUNT
    spardl.workspace_init(st.ws, P, P, n, kb)
    assert spardl.ws_error(st.ws) == 0
    st.residual_add(grad)
    st.block_topk()
    assert spardl.ws_error(st.ws) == 0


def test_invalid_arguments_raise():
    st = spardl.SparDLStep(4, 4000, 10)
    with pytest.raises(spardl.SpardlError):
        spardl.sparse_merge_topk(st.sp_idx, st.sp_val, 4, 4000, 10, 3, st.drop_idx[0], st.drop_val[0],
                                 st.drop_cnt[0], st.ws)
    with pytest.raises(spardl.SpardlError):
        spardl.block_topk(st.acc, 4, 4000, 4, 1001, st.sp_idx, st.sp_val, None, st.ws)
    small = st.ws[:1024]
    with pytest.raises(spardl.SpardlError) as e:
        spardl.block_topk(st.acc, 4, 4000, 4, 10, st.sp_idx, st.sp_val, None, small)
    assert e.value.status == spardl.ECAPACITY
