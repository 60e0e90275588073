"""Lane layouts of the gather kernels at the widths and shapes where they change,
against the oracle."""
import numpy as np
import pytest
import torch

import synth
import test_gpu_parity
from test_gpu_parity import (check_dense_matmul, check_mlp, check_sddmm, check_softmax,
                             check_softmax_backward,
                             check_sddmm_softmax, check_sddmm_softmax_backward, check_spmm, dev, host,
                             say)

pytestmark = pytest.mark.gpu

fg = None  # imported lazily so that collection works without the library


def setup_module(module):
    global fg
    test_gpu_parity.setup_module(test_gpu_parity)  # its check functions call the package
    fg = test_gpu_parity.fg


def _graph(seed, n, m, lo, hi):
    """n rows of lo .. hi - 1 sources out of m, one of them empty; the edge
    count is no multiple of 4."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(lo, hi, size=n)
    deg[n // 2] = 0
    deg[-1] += (1 - deg.sum()) % 4
    dst = np.repeat(np.arange(n), deg).astype(np.int64)
    return synth.coo_to_csr(dst, rng.integers(0, m, size=dst.size).astype(np.int64), n, m)


@pytest.mark.parametrize("d", [4, 5, 7, 15, 17, 31, 33, 66, 101, 41, 63, 65, 126, 129, 255, 257, 300, 383, 385,
                               511, 513, 767, 768, 769, 1023, 1025, 2049])
def test_ragged_rows(d):
    """Widths around every layout's edge, most of them no multiple of 4, with
    64-edge and 256-edge batches, whole and split rows."""
    rng = np.random.default_rng(d)
    for lo, hi, segment in ((0, 5, 0), (0, 40, 0), (130, 420, 0), (130, 420, 100)):
        csr = _graph(d + lo, 40, 90, lo, hi)
        G = fg.Graph.from_csr(csr)
        x = rng.standard_normal((csr.num_cols, d)).astype(np.float32)
        xd = rng.standard_normal((csr.num_rows, d)).astype(np.float32)
        w = rng.random(csr.nnz, dtype=np.float32)
        for plan in (None, fg.Plan(G, d, segment_edges=segment)):
            check_spmm(csr, G, x, plan=plan)
            check_spmm(csr, G, x, plan=plan, edge=w)
            check_spmm(csr, G, x, plan=plan, reduce="max")
            check_spmm(csr, G, x, plan=plan, edge=w, reduce="max")
            check_sddmm(csr, G, x, xd, plan=plan)


@pytest.mark.parametrize("heads,dh", [(2, 3), (3, 5), (8, 6), (16, 10), (17, 3), (20, 4), (40, 7),
                                      (33, 8), (2, 129), (24, 30)])
def test_ragged_heads(heads, dh):
    """Heads that straddle a lane's four floats, up to and above the heads
    whose weights a wavefront stages in LDS."""
    for lo, hi, segment in ((0, 90, 30), (100, 300, 90)):  # scalar lanes; float4 lanes
        csr = _graph(heads, 60, 50, lo, hi)
        G = fg.Graph.from_csr(csr)
        rng = np.random.default_rng(dh)
        x = rng.standard_normal((csr.num_cols, heads, dh)).astype(np.float32)
        w = rng.standard_normal((csr.nnz, heads)).astype(np.float32)
        for plan in (None, fg.Plan(G, heads * dh, segment_edges=segment)):
            for reduce in ("sum", "max"):
                check_spmm(csr, G, x, plan=plan, edge=w, heads=heads, reduce=reduce)


def test_ragged_mlp():
    rng = np.random.default_rng(3)
    for hi in (300, 9):  # short rows: scalar lanes
        csr = _graph(3, 50, 70, 0, hi)
        G = fg.Graph.from_csr(csr)
        xs = rng.standard_normal((csr.num_cols, 8)).astype(np.float32)
        xd = rng.standard_normal((csr.num_rows, 8)).astype(np.float32)
        for d_out in (5, 37, 67, 130):
            w = rng.standard_normal((8, d_out)).astype(np.float32)
            for plan in (None, fg.Plan(G, d_out, segment_edges=70), fg.Plan(G, d_out, segment_edges=4)):
                check_mlp(csr, G, xs, xd, w, plan=plan)


@pytest.mark.parametrize("d", [6, 41, 130, 601])
def test_ragged_tail_infinities(d):
    """A tail lane repeats its neighbour's floats: an infinity there counts
    once (times 0 it would be NaN), and a NaN stays in its own column."""
    csr = _graph(d, 30, 40, 1, 50)
    G = fg.Graph.from_csr(csr)
    rng = np.random.default_rng(d)
    x = rng.standard_normal((csr.num_cols, d)).astype(np.float32)
    xd = (rng.random((csr.num_rows, d)) + 0.5).astype(np.float32)
    for k in range(1, 6):
        x[k, d - k] = np.inf
    say("infinities in the last columns, d=%d" % d)
    s = host(fg.gsddmm(G, dev(x), dev(xd)))
    rows = synth.csr_rows(csr)
    ref = (x[csr.indices].astype(np.float64) * xd[rows]).sum(1)
    np.testing.assert_array_equal(np.isposinf(s), np.isposinf(ref))
    assert not np.isnan(s).any()
    x[7, d - 2] = np.nan
    y = host(fg.gspmm(G, dev(x)))
    ref = np.zeros((csr.num_rows, d))
    np.add.at(ref, rows, x[csr.indices].astype(np.float64))
    np.testing.assert_array_equal(np.isnan(y), np.isnan(ref))


@pytest.mark.parametrize("n,d_in,d_out", [(1, 15, 3), (63, 16, 63), (64, 17, 64), (65, 33, 65),
                                          (129, 32, 128), (200, 31, 129), (70405, 17, 65),
                                          (70405, 3, 130), (35300, 48, 256), (1, 1, 1), (65537, 12, 64),
                                          (65536, 13, 3), (70001, 5, 100), (70001, 8, 129),
                                          (70405, 33, 7), (65549, 24, 16), (65549, 40, 1)])
def test_dense_tiles(n, d_in, d_out):
    """Tile and step edges of the matrix-core transform; from 1024 tiles of
    64 x 128 on its wider tiles, and few columns of X without staging."""
    check_dense_matmul(n, d_in, d_out, n + d_in)
    check_dense_matmul(n, d_in, d_out, n + d_out, exact=True)


@pytest.mark.parametrize("heads,dh", [(2, 4), (8, 8), (8, 6), (3, 5), (17, 4), (33, 8), (5, 20),
                                      (2, 33), (3, 64), (9, 12), (2, 129), (2, 256), (2, 258),
                                      (4, 3), (70, 2)])
def test_sddmm_head_layouts(heads, dh):
    """Heads of every lane count, idle lanes in a head, tails that overlap
    their neighbour, head counts over several passes, and the shapes left to
    scalar lanes; with edge ids as well."""
    rng = np.random.default_rng(heads * 1000 + dh)
    for lo, hi in ((0, 30), (60, 200)):
        csr = _graph(dh, 40, 60, lo, hi)
        x = rng.standard_normal((csr.num_cols, heads, dh)).astype(np.float32)
        xd = rng.standard_normal((csr.num_rows, heads, dh)).astype(np.float32)
        G = fg.Graph.from_csr(csr)
        for plan in (None, fg.Plan(G, heads * dh, segment_edges=50)):
            check_sddmm(csr, G, x, xd, plan=plan, heads=heads)
        csc = synth.csr_to_csc(csr)
        Gt = fg.Graph.from_csr(csc, nnz_total=csr.nnz)
        check_sddmm(csc, Gt, xd, x, plan=fg.Plan(Gt, heads * dh), heads=heads, nnz_total=csr.nnz)


@pytest.mark.parametrize("dh", [6, 8])
def test_sddmm_head_infinities(dh):
    """An infinity in a head's last features counts once and in that head."""
    csr = _graph(5, 30, 40, 1, 50)
    rng = np.random.default_rng(dh)
    x = rng.standard_normal((csr.num_cols, 3, dh)).astype(np.float32)
    xd = (rng.random((csr.num_rows, 3, dh)) + 0.5).astype(np.float32)
    for k in range(1, 6):
        x[k, k % 3, dh - k] = np.inf
    s = host(fg.gsddmm(fg.Graph.from_csr(csr), dev(x), dev(xd)))
    ref = (x[csr.indices].astype(np.float64) * xd[synth.csr_rows(csr)]).sum(-1)
    np.testing.assert_array_equal(np.isposinf(s), np.isposinf(ref))
    assert not np.isnan(s).any()


@pytest.mark.parametrize("heads,dh", [(8, 8), (4, 4), (16, 8), (16, 4), (3, 8), (2, 4)])
def test_score_gradient_narrow_heads(heads, dh):
    csr = _graph(heads, 60, 60, 0, 150)
    G = fg.Graph.from_csr(csr)
    rng = np.random.default_rng(dh)
    x = rng.integers(-3, 4, (csr.num_cols, heads, dh)).astype(np.float32)
    dy = rng.integers(-3, 4, (csr.num_rows, heads, dh)).astype(np.float32)
    s = (3 * rng.standard_normal((csr.nnz, heads))).astype(np.float32)
    for plan in (None, fg.Plan(G, heads * dh), fg.Plan(G, heads * dh, segment_edges=64)):
        for leaky in (True, False):
            check_sddmm_softmax_backward(csr, G, x, dy, s, plan=plan, leaky=leaky)


@pytest.mark.parametrize("dh", [4, 8, 16])
def test_score_gradient_twelve_heads(dh):
    """Twelve heads: a multiple of four that does not divide a wavefront's 256
    values, so that no lane keeps its heads along a row."""
    csr = _graph(dh, 60, 60, 0, 150)
    G = fg.Graph.from_csr(csr)
    rng = np.random.default_rng(dh)
    x = rng.integers(-3, 4, (csr.num_cols, 12, dh)).astype(np.float32)
    dy = rng.integers(-3, 4, (csr.num_rows, 12, dh)).astype(np.float32)
    s = (3 * rng.standard_normal((csr.nnz, 12))).astype(np.float32)
    for plan in (None, fg.Plan(G, 12 * dh), fg.Plan(G, 12 * dh, segment_edges=64)):
        for leaky in (True, False):
            check_sddmm_softmax_backward(csr, G, x, dy, s, plan=plan, leaky=leaky)


@pytest.mark.parametrize("d", [4, 16, 20, 32, 64, 128, 256, 512, 1024])
def test_fused_scores_and_softmax(d):
    """One pass for scores and weights on plans of short items and without a
    plan: full and masked steps of every layout, whole and split rows."""
    rng = np.random.default_rng(d)
    csr = _graph(d, 70, 60, 0, 80)
    G = fg.Graph.from_csr(csr)
    x = (rng.standard_normal((csr.num_cols, d)) / d ** 0.25).astype(np.float32)
    xd = (rng.standard_normal((csr.num_rows, d)) / d ** 0.25).astype(np.float32)
    for plan in (None, fg.Plan(G, d, segment_edges=33)):
        check_sddmm_softmax(csr, G, x, xd, plan=plan)
        check_sddmm_softmax(csr, G, x, xd, plan=plan, leaky=False)


@pytest.mark.parametrize("d", [16, 32, 48, 64, 96, 128])
def test_repeated_edges(d):
    """Graphs that repeat many edges: batches packed to one entry per run of
    copies, in every layout, with runs across lanes and batches, whole and
    split rows, ties, and edge ids; and the same plan after the sources were
    reordered so that no copies are neighbours."""
    rng = np.random.default_rng(d)
    n, m = 200, 90
    deg = rng.integers(200, 900, size=n)
    deg[3] = 0
    dst = np.repeat(np.arange(n), deg).astype(np.int64)
    src = (m * rng.random(dst.size) ** 3).astype(np.int64)  # runs of 1 to 200 copies
    src[: deg[0]] = 7  # one run over several batches
    csr = synth.coo_to_csr(dst, src, n, m)
    ew = (rng.random(csr.nnz) + 0.01).astype(np.float32)
    ewi = rng.integers(1, 4, csr.nnz).astype(np.float32)
    x = rng.standard_normal((m, d)).astype(np.float32)
    xi = rng.integers(-4, 5, (m, d)).astype(np.float32)
    xd = rng.standard_normal((n, d)).astype(np.float32)
    assert np.mean(csr.indices[1:] == csr.indices[:-1]) > 0.5

    def check(csr, G, plan):
        check_spmm(csr, G, x, plan=plan)
        check_spmm(csr, G, xi, plan=plan, exact=True)
        check_spmm(csr, G, x, plan=plan, edge=ew)
        check_spmm(csr, G, xi, plan=plan, edge=ewi, exact=True)
        check_spmm(csr, G, x, plan=plan, reduce="max")
        check_spmm(csr, G, xi, plan=plan, reduce="max")
        check_spmm(csr, G, x, plan=plan, edge=ew, reduce="max")
        check_sddmm(csr, G, x, xd, plan=plan)

    G = fg.Graph.from_csr(csr)
    for segment in (0, 300):
        check(csr, G, _merging_plan(G, d, segment))
    w = rng.standard_normal((8, d)).astype(np.float32)
    check_mlp(csr, G, rng.standard_normal((m, 8)).astype(np.float32),
              rng.standard_normal((n, 8)).astype(np.float32), w, plan=fg.Plan(G, d))
    csc = synth.csr_to_csc(csr)
    Gt = fg.Graph.from_csr(csc, nnz_total=csr.nnz)
    plan = fg.Plan(Gt, d)
    check_sddmm(csc, Gt, xd, x, plan=plan, nnz_total=csr.nnz)
    check_spmm(csc, Gt, xd, plan=plan, nnz_total=csr.nnz)
    check_spmm(csc, Gt, xd, plan=plan, edge=ew, reduce="max", nnz_total=csr.nnz)
    # the plan's hint outlives the order of the sources
    mixed = csr.indices.copy()
    for r in range(n):
        rng.shuffle(mixed[csr.indptr[r]:csr.indptr[r + 1]])
    plan = fg.Plan(G, d, source_slab_rows=-2)
    G.indices.copy_(dev(mixed))
    plan.validate()
    check(synth.CSR(n, m, csr.indptr, mixed), G, plan)


def _merging_plan(G, d, segment):
    """A plan on which the gather kernels merge repeated edges (the layouts of
    65 to 128 floats take their wide batches from 112 edges an item on)."""
    plan = fg.Plan(G, d, segment_edges=segment)
    info = plan.info()
    assert info["merges_repeats"] and G.nnz >= 112 * info["num_segments"]
    return plan


def test_repeated_edges_infinities():
    """Copies of an infinite or NaN source stay what repeated adds give."""
    n, m, d = 128, 20, 128
    rng = np.random.default_rng(0)
    dst = np.repeat(np.arange(n), 300).astype(np.int64)
    csr = synth.coo_to_csr(dst, rng.integers(0, m, dst.size).astype(np.int64), n, m)
    x = rng.standard_normal((m, d)).astype(np.float32)
    x[3, 5], x[4, 6], x[5, 7] = np.inf, -np.inf, np.nan
    G = fg.Graph.from_csr(csr)
    plan = _merging_plan(G, d, 300)
    y = host(fg.gspmm(G, dev(x), plan=plan))
    with np.errstate(invalid="ignore"):
        ref = np.zeros((n, d))
        np.add.at(ref, synth.csr_rows(csr), x[csr.indices].astype(np.float64))
    np.testing.assert_array_equal(np.isnan(y), np.isnan(ref))
    np.testing.assert_array_equal(np.isinf(y), np.isinf(ref))
    fin = np.isfinite(ref)
    np.testing.assert_allclose(y[fin], ref[fin], rtol=2e-5, atol=2e-4)


@pytest.mark.parametrize("more", [0, 40])
@pytest.mark.parametrize("heads,batches", [(8, 6), (4, 12)])
def test_score_gradient_row_lengths(heads, batches, more):
    """Rows around the longest whose gradients stay in registers (6 batches of
    64 edges with 8 heads, 12 with 4), and around one batch; the register form
    runs where rows that it holds have three quarters of the edges (more)."""
    rng = np.random.default_rng(heads)
    top = 64 * batches
    deg = np.array([0, 1, 63, 64, 65, 128, top - 1, top, top + 1, top + 64, 2 * top, 3])
    deg = np.concatenate([deg, np.full(more, top)])
    assert (4 * deg[deg <= top].sum() >= 3 * deg.sum()) == (more > 0)
    n = deg.size
    dst = np.repeat(np.arange(n), deg).astype(np.int64)
    csr = synth.coo_to_csr(dst, rng.integers(0, 50, dst.size).astype(np.int64), n, 50)
    G = fg.Graph.from_csr(csr)
    plan = fg.Plan(G, heads * 16, segment_edges=16384)
    assert plan.info()["plain_slots"] == 0
    x = rng.integers(-3, 4, (50, heads, 16)).astype(np.float32)
    dy = rng.integers(-3, 4, (n, heads, 16)).astype(np.float32)
    s = (3 * rng.standard_normal((csr.nnz, heads))).astype(np.float32)
    for leaky in (True, False):
        check_sddmm_softmax_backward(csr, G, x, dy, s, plan=plan, leaky=leaky)


@pytest.mark.parametrize(
    "w", [(1.0, -2.0), (0.0, 1.0), (2.0**127, 2.0**127), (np.inf, -np.inf), (-1.0, -2.0)])
@pytest.mark.parametrize("d", [72, 128])
def test_repeated_edges_weights(d, w):
    """Weighted copies of an edge to infinite, NaN, zero and small features: what
    adding them one by one gives, where their weights have two signs, a zero or
    a sum that overflows as where they have one sign."""
    n, m = 128, 16
    dst = np.repeat(np.arange(n), 512).astype(np.int64)
    csr = synth.coo_to_csr(dst, np.tile(np.repeat(np.arange(m), 32), n).astype(np.int64), n, m)
    assert np.mean(csr.indices[1:] == csr.indices[:-1]) > 0.5
    x = np.full((m, d), 2.0**-40, np.float32)  # 32 copies of 2^127 2^-40 stay finite
    x[3, 5], x[4, 6], x[5, 7], x[:, 8], x[3, d - 1] = np.inf, -np.inf, np.nan, 0, np.inf
    ew = np.full(csr.nnz, 0.5, np.float32)
    ew[100:102] = ew[1000:1002] = ew[1535:1537] = ew[130:132] = ew[163:165] = w
    G = fg.Graph.from_csr(csr)
    y = host(fg.gspmm(G, dev(x), dev(ew), msg="src_mul_edge", plan=_merging_plan(G, d, 512)))
    ref = np.zeros((n, d))
    with np.errstate(invalid="ignore"):
        np.add.at(ref, synth.csr_rows(csr),
                  x[csr.indices].astype(np.float64) * ew[:, None].astype(np.float64))
    np.testing.assert_array_equal(np.isnan(y), np.isnan(ref))
    np.testing.assert_array_equal(np.isinf(y), np.isinf(ref))
    fin = np.isfinite(ref)
    # 512 float sums of one-signed terms, or of two terms against the rest
    np.testing.assert_allclose(y[fin], ref[fin], rtol=512 * 2.0**-24, atol=512 * 2.0**-24 * 2.0**-30)


def _run_sums(keys, w):
    """Weights of each run of equal keys in a batch of 256 edges, added as the
    kernel states it: four neighbouring edges in order, then lanes by steps of
    1, 2, 4, ... (float32)."""
    f = np.float32
    start = np.r_[True, keys[1:] != keys[:-1]]
    head = start.reshape(64, 4)
    part = w.reshape(64, 4).astype(f).copy()
    for q in range(1, 4):
        part[:, q] = np.where(head[:, q], part[:, q], f(part[:, q - 1] + part[:, q]))
    starts = head.any(1)
    back = np.array([next(b for b in range(64) if starts[l - b]) for l in range(64)])
    t = part[:, 3].copy()
    for d in (1, 2, 4, 8, 16, 32):
        o = np.r_[np.zeros(d, f), t[:-d]]
        t = np.where(back >= d, f(o + t), t)
    before = np.r_[f(0), t[:-1]]
    whole = np.logical_or.accumulate(head, axis=1)
    part = np.where(whole, part, f(before[:, None] + part))
    return keys[start], part.reshape(-1)[np.r_[np.nonzero(start)[0][1:] - 1, 255]]


@pytest.mark.parametrize("d", [72, 128])
def test_repeated_edges_order(d):
    """The weights of an edge's copies are added in the order that the kernel
    states, whatever the hardware does: with unit features of one column per
    source, each output is one run's sum, bit for bit, on every call."""
    rng = np.random.default_rng(d)
    n, m = 128, d
    src = np.concatenate([np.sort(rng.integers(0, rng.integers(1, m + 1), 256)) for _ in range(n)])
    csr = synth.coo_to_csr(np.repeat(np.arange(n), 256).astype(np.int64), src.astype(np.int64), n, m)
    w = (rng.random(csr.nnz) + 0.01).astype(np.float32)
    want = np.zeros((n, m), np.float32)
    for r in range(n):
        k, v = _run_sums(csr.indices[256 * r:256 * r + 256], w[256 * r:256 * r + 256])
        want[r, k] = v
    G = fg.Graph.from_csr(csr)
    plan = _merging_plan(G, d, 256)
    x, w = dev(np.eye(m, dtype=np.float32)), dev(w)
    for _ in range(3):
        y = host(fg.gspmm(G, x, w, msg="src_mul_edge", plan=plan))
        np.testing.assert_array_equal(y, want)
    # rows in pieces, any features: call to call, and without allocation
    plan = _merging_plan(G, d, 150)
    x = dev(rng.standard_normal((m, d)).astype(np.float32))
    y = host(fg.gspmm(G, x, w, msg="src_mul_edge", plan=plan))
    out = dev(np.zeros((n, d), np.float32))
    for _ in range(3):
        np.testing.assert_array_equal(host(fg.gspmm(G, x, w, msg="src_mul_edge", plan=plan)), y)
        fg.gspmm_noalloc(G, x, out, edge=w, msg="src_mul_edge", plan=plan)
        np.testing.assert_array_equal(host(out), y)


@pytest.mark.parametrize("deg,long_row,segment,two_pass", [(100, 3000, 1000, True),
                                                           (40, 1000, 0, False)])
def test_scores_and_softmax_small_weights(deg, long_row, segment, two_pass):
    """Weights of e^-80 to 1 to a few units in the last place, whichever route
    the call takes: as two operators on plans of 56 edges an item and more, and
    for rows that a plan's shorter pieces cut.  Integer scores, so that only the
    exponentials, the sum and its reciprocal round: expf to one ulp (2 units of
    2^-24), the reciprocal and the product half an ulp each, and the sum half an
    ulp an addition (two a lane and six over the lanes for 128 edges, 24 and a
    merge of three for the long row)."""
    rng = np.random.default_rng(deg)
    n, m, d = 200, 81, 128
    counts = np.full(n, deg)
    counts[7] = long_row
    dst = np.repeat(np.arange(n), counts).astype(np.int64)
    src = rng.integers(0, m, dst.size).astype(np.int64)
    src[np.r_[0, np.cumsum(counts)[:-1]]] = 0  # a score of 0 in every row
    csr = synth.coo_to_csr(dst, src, n, m)
    x = np.zeros((m, d), np.float32)
    x[:, 3] = -np.arange(m)
    xd = np.ones((n, d), np.float32)
    G = fg.Graph.from_csr(csr)
    plan = fg.Plan(G, d, segment_edges=segment)
    info = plan.info()
    assert info["num_split_rows"] == 1
    assert (csr.nnz >= 56 * info["num_segments"]) == two_pass
    s, a = fg.gsddmm_edge_softmax(G, dev(x), dev(xd), leaky=False, plan=plan)
    np.testing.assert_array_equal(host(s), -csr.indices.astype(np.float32))
    e = np.exp(-csr.indices.astype(np.float64))
    rows = synth.csr_rows(csr)
    ref = e / np.bincount(rows, e, n)[rows]
    err = np.abs(host(a) / ref - 1)
    short = rows != 7
    assert err[short].max() <= 16 * 2.0**-24, err[short].max()
    assert err[~short].max() <= 36 * 2.0**-24, err[~short].max()


@pytest.mark.parametrize("heads,dh", [(1, 16), (4, 32), (2, 128)])
def test_attention_split_rows_divide(heads, dh):
    """A split row's output is its weighted sum over its exponential sum, in one
    rounding: with equal scores and equal features both sums are exact and the
    quotient is the feature itself (49 times the rounded 1/49 is not 1)."""
    n = 80
    counts = np.arange(n) * 7 + 41  # 49, 98, 196, ... among them
    dst = np.repeat(np.arange(n), counts).astype(np.int64)
    csr = synth.coo_to_csr(dst, np.arange(dst.size) % 30, n, 30)
    G = fg.Graph.from_csr(csr)
    plan = fg.Plan(G, heads * dh, segment_edges=20, item_order=1)
    assert plan.info()["num_split_rows"] == n
    x = dev(np.full((30, heads, dh), 3.0, np.float32))
    xd = dev(np.zeros((n, heads, dh), np.float32))
    say("attention over equal scores, H=%d dh=%d" % (heads, dh))
    np.testing.assert_array_equal(host(fg.gat_aggregate(G, x, xd, plan=plan)),
                                  np.full((n, heads, dh), 3.0, np.float32))


def test_results_are_plain_tensors():
    """Inputs of a tensor subclass give plain tensors."""
    class Sub(torch.Tensor):
        pass

    csr = _graph(1, 20, 20, 0, 9)
    G = fg.Graph.from_csr(csr)
    x = dev(np.ones((20, 4), np.float32)).as_subclass(Sub)
    for y in (fg.gspmm(G, x), fg.gsddmm(G, x, x), fg.gat_aggregate(G, x, x)):
        assert type(y) is torch.Tensor


@pytest.mark.parametrize("share", [0.0, 0.5])
def test_repeats_hint(share):
    """Whether a plan merges repeated edges depends on the graph alone: not on
    the item order asked for, nor on host copies of the indices."""
    rng = np.random.default_rng(3)
    n = 100
    src = np.stack([rng.permutation(400)[:60] for _ in range(n)]).astype(np.int64)
    src = np.concatenate([src, src[:, :int(60 * share)]], axis=1)
    csr = synth.coo_to_csr(np.repeat(np.arange(n), src.shape[1]).astype(np.int64), src.reshape(-1),
                           n, 400)
    G = fg.Graph.from_csr(csr)
    D = fg.Graph(n, 400, G.indptr, G.indices)  # no host copies
    assert G.indices_host is not None and D.indices_host is None
    for g in (G, D):
        for order in (0, 1, 2, 3):
            assert fg.Plan(g, 32, item_order=order).info()["merges_repeats"] == (share > 0)


@pytest.mark.parametrize("d", [72, 128])
def test_repeated_edges_subnormal_weights(d):
    """Copies whose weights are subnormal keep every bit: integers of 2^-149
    times features of 2^100, with sums below 2^24, are exact."""
    n, m = 128, 16
    rng = np.random.default_rng(d)
    dst = np.repeat(np.arange(n), 256).astype(np.int64)
    csr = synth.coo_to_csr(dst, rng.integers(0, m, dst.size).astype(np.int64), n, m)
    k = rng.integers(1, 4096, csr.nnz)
    G = fg.Graph.from_csr(csr)
    x = np.full((m, d), 2.0**100, np.float32)
    y = host(fg.gspmm(G, dev(x), dev(np.ldexp(k.astype(np.float64), -149).astype(np.float32)),
                      msg="src_mul_edge", plan=_merging_plan(G, d, 256)))
    want = np.ldexp(np.bincount(synth.csr_rows(csr), k, n), -49)[:, None] * np.ones(d)
    np.testing.assert_array_equal(y.astype(np.float64), want)


@pytest.mark.parametrize("heads,dh", [(1, 128), (4, 32), (8, 4)])
@pytest.mark.parametrize("segment", [0, 40])
def test_attention_nan_and_infinite_scores(heads, dh, segment):
    """A NaN or an infinite score makes its row's head NaN and leaves the other
    rows and heads alone, in whole rows and in split ones, wherever it stands."""
    rng = np.random.default_rng(dh)
    n, m = 70, 300
    src = np.stack([np.sort(rng.permutation(m)[:90]) for _ in range(n)]).astype(np.int64)
    csr = synth.coo_to_csr(np.repeat(np.arange(n), 90).astype(np.int64), src.reshape(-1), n, m)
    G = fg.Graph.from_csr(csr)
    plan = fg.Plan(G, heads * dh, segment_edges=segment)
    x = rng.standard_normal((m, heads, dh)).astype(np.float32)
    xd = (rng.random((n, heads, dh)) + 0.5).astype(np.float32)
    clean = host(fg.gat_aggregate(G, dev(x), dev(xd), plan=plan))
    assert np.isfinite(clean).all()
    x[11, 0, 1], x[200, heads - 1, 2] = np.nan, np.inf
    y = host(fg.gat_aggregate(G, dev(x), dev(xd), plan=plan))
    hit = np.zeros((n, heads), bool)
    hit[:, 0] |= (src == 11).any(1)
    hit[:, heads - 1] |= (src == 200).any(1)
    assert hit.any(0)[[0, heads - 1]].all() and not hit.all()
    assert np.isnan(y[hit]).all()
    np.testing.assert_array_equal(y[~hit], clean[~hit])


@pytest.mark.parametrize("heads", [1, 2, 4, 5, 8])
def test_softmax_cut_rows_taken_whole(heads):
    """Plans that cut rows by themselves: with few values a row the softmax and
    its backward take the rows whole (700 edges with up to 5 heads), with more
    in pieces; the score gradient runs as one pass where no row outlasts the
    rest (nnz / 2048 edges), else as two operators.  With edge ids as well."""
    rng = np.random.default_rng(heads)
    for n, rest in ((300, 20), (15000, 96)):
        deg = rng.integers(rest // 2, rest + rest // 2, n)
        deg[5], deg[n - 2], deg[9] = 700, 513, 0
        dst = np.repeat(np.arange(n), deg).astype(np.int64)
        csr = synth.coo_to_csr(dst, rng.integers(0, 500, dst.size).astype(np.int64), n, 500)
        G = fg.Graph.from_csr(csr)
        plan = fg.Plan(G, heads * 4)
        assert plan.info()["plain_slots"] >= 2
        rows = np.r_[0:12, n // 2, n - 3:n]
        s = (3 * rng.standard_normal((csr.nnz, heads))).astype(np.float32)
        go = rng.standard_normal((csr.nnz, heads)).astype(np.float32)
        for leaky in (True, False):
            check_softmax(csr, G, s, rows=rows, plan=plan, heads=heads, leaky=leaky)
            check_softmax_backward(csr, G, s, go, rows=rows, plan=plan, heads=heads, leaky=leaky)
            if heads > 1:
                x = rng.integers(-3, 4, (500, heads, 4)).astype(np.float32)
                dy = rng.integers(-3, 4, (n, heads, 4)).astype(np.float32)
                check_sddmm_softmax_backward(csr, G, x, dy, s, plan=plan, leaky=leaky, rows=rows)
    csc = synth.csr_to_csc(csr)
    deg = csc.degrees()
    Gt = fg.Graph.from_csr(csc, nnz_total=csr.nnz)
    plan = fg.Plan(Gt, heads * 4)
    assert plan.info()["plain_slots"] >= 2 and deg.max() > 2000
    rows = np.r_[0:5, deg.argmax()]
    check_softmax(csc, Gt, s, rows=rows, plan=plan, heads=heads, nnz_total=csr.nnz)
    check_softmax_backward(csc, Gt, s, go, rows=rows, plan=plan, heads=heads, nnz_total=csr.nnz)
