"""GPU parity of the individual steps against the fp64 oracle, through the C ABI.

Integer / index work (CSR build, degrees, dinv, nonzero counts, compressed
feature views) must match bit for bit; fp32 results must stay within 1e-4 of
the oracle relative to each element's magnitude scale (sum of |terms|).
"""
import ctypes as C

import numpy as np
import pytest
import torch

import gcn_synth as gs
from helpers import adversarial_graphs, assert_mag_close, assert_norm_close, messy, note

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_2512_01678_amd.gcn as G
    return G


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy()


def pitched(a, ld):
    """Device copy of a (rows x w) with row pitch ld (extra columns filled with NaN)."""
    rows, w = a.shape
    buf = torch.full((rows, ld), float("nan"), dtype=torch.float32, device="cuda")
    buf[:, :w] = dev(a.astype(np.float32))
    return buf[:, :w]


# ---------------------------------------------------------------------------
# a1: A + I in CSR
# ---------------------------------------------------------------------------


def check_graph_equal(dg, og, n):
    assert dg.nnz == og.nnz
    np.testing.assert_array_equal(host(dg.row_ptr), og.row_ptr)
    np.testing.assert_array_equal(host(dg.col_idx)[:og.nnz], og.col_idx)
    np.testing.assert_array_equal(host(dg.deg)[:n], og.deg)
    np.testing.assert_array_equal(host(dg.dinv)[:n].view(np.int32), og.dinv.view(np.int32))
    # stored entries of A_hat: fl32(dinv[i] * dinv[j]), one IEEE rounding
    rows = np.repeat(np.arange(n), np.diff(og.row_ptr))
    want = og.dinv[rows] * og.dinv[og.col_idx]
    assert want.dtype == np.float32
    np.testing.assert_array_equal(host(dg.val)[:og.nnz].view(np.int32), want.view(np.int32))


@pytest.mark.parametrize("case", adversarial_graphs(), ids=lambda c: c[0])
def test_build_csr_bit_exact(G, orc, case):
    name, n, s, d = case
    print(f"[csr] {name} n={n} edges={s.size}", flush=True)
    check_graph_equal(G.build_csr(n, dev(s), dev(d)), orc.build_csr(n, s, d), n)


@pytest.mark.parametrize("name", ["cora_like", "arxiv_like"])
def test_build_csr_workloads(G, orc, name):
    wl = gs.WORKLOADS[name]
    s, d = gs.make_graph(wl)
    print(f"[csr] {name} n={wl.n} edges={s.size}", flush=True)
    check_graph_equal(G.build_csr(wl.n, dev(s), dev(d)), orc.build_csr(wl.n, s, d), wl.n)


def test_build_csr_rmat_small(G, orc):
    s, d = gs.rmat(14, 1 << 18)
    check_graph_equal(G.build_csr(1 << 14, dev(s), dev(d)), orc.build_csr(1 << 14, s, d), 1 << 14)


def test_build_csr_rejects_out_of_range(G):
    s = np.array([0, 1, 5], np.int32)
    d = np.array([1, 2, 0], np.int32)
    with pytest.raises(G.GcnError) as ei:
        G.build_csr(5, dev(s), dev(d))
    assert ei.value.status == G.E_RANGE
    with pytest.raises(G.GcnError):
        G.build_csr(5, dev(np.array([-1], np.int32)), dev(np.array([0], np.int32)))


# ---------------------------------------------------------------------------
# a2: density probe, decision, X_csr / X_csc
# ---------------------------------------------------------------------------


def feature_cases():
    rng = np.random.default_rng(77)
    special = rng.standard_normal((50, 70)).astype(np.float32)
    special[rng.random((50, 70)) < 0.6] = 0.0
    special[3, 4] = -0.0
    special[5, 6] = np.nan
    special[7, 8] = np.inf
    special[9, :] = 0.0
    thr = np.zeros((40, 25), np.float32)
    thr.flat[: 40 * 25 // 5] = 1.5
    rng.shuffle(thr.reshape(-1))
    return [
        ("cora_like", gs.make_features(gs.WORKLOADS["cora_like"])),
        ("nonneg10", gs.features_bernoulli(2500, 4096, 0.1, binary=False)),
        ("nonneg0.1", gs.features_bernoulli(3000, 1000, 0.001, binary=False)),
        ("special", special),
        ("zeros", np.zeros((33, 17), np.float32)),
        ("ones", np.ones((33, 17), np.float32)),
        ("identity", np.eye(64, 40, dtype=np.float32)),
        ("threshold", thr),
        ("one_col", (rng.random((1100, 1)) < 0.5).astype(np.float32)),
        ("f65", (rng.random((2100, 65)) < 0.2).astype(np.float32) * 2.0),
    ]


@pytest.mark.parametrize("case", feature_cases(), ids=lambda c: c[0])
def test_feature_stats_bit_exact(G, orc, case):
    name, X = case
    n, f = X.shape
    print(f"[features] {name} {n}x{f}", flush=True)
    nnz, rn = orc.feature_counts(X)
    mode = orc.sparse_decision(nnz, n, f)
    Xd = pitched(X, G.pitch(f) + 4)
    rnd = torch.zeros(n, dtype=torch.int64, device="cuda")
    info, sx = G.feature_stats(Xd, tau=(4, 5), materialize=True, row_nnz=rnd)
    assert info["nnz"] == nnz and info["mode"] == mode
    assert info["sparsity"] == pytest.approx(orc.sparsity(nnz, n, f), abs=1e-15)
    np.testing.assert_array_equal(host(rnd), rn)
    rp, col, val = orc.dense_to_csr(X)
    np.testing.assert_array_equal(host(sx.row_ptr), rp)
    np.testing.assert_array_equal(host(sx.col)[:nnz], col)
    np.testing.assert_array_equal(host(sx.val)[:nnz].view(np.int32), val.view(np.int32))
    cp, row, cval = orc.dense_to_csc(X)
    np.testing.assert_array_equal(host(sx.col_ptr), cp)
    np.testing.assert_array_equal(host(sx.row)[:nnz], row)
    np.testing.assert_array_equal(host(sx.cval)[:nnz].view(np.int32), cval.view(np.int32))


def test_feature_decision_tau_and_force(G, orc):
    X = np.zeros((40, 25), np.float32)
    X.flat[: 40 * 25 // 5 + 1] = 1.0
    info, _ = G.feature_stats(dev(X), tau=(4, 5), materialize=False)
    assert info["mode"] == G.DENSE
    info, _ = G.feature_stats(dev(X), tau=(3, 4), materialize=False)
    assert info["mode"] == G.SPARSE
    info, _ = G.feature_stats(dev(X), force_mode=G.SPARSE, materialize=False)
    assert info["mode"] == G.SPARSE
    # the default threshold, measured on this GPU: tau = 15/16, sparse iff nnz <= N F / 16
    assert G.TAU_MI355X == (15, 16)
    Y = np.zeros((64, 50), np.float32)
    Y.flat[: 64 * 50 // 16] = 2.0
    info, _ = G.feature_stats(dev(Y), materialize=False)
    assert info["mode"] == G.SPARSE and orc.sparse_decision(info["nnz"], 64, 50, 15, 16) == G.SPARSE
    Y.flat[64 * 50 // 16] = 2.0
    info, _ = G.feature_stats(dev(Y), materialize=False)
    assert info["mode"] == G.DENSE and orc.sparse_decision(info["nnz"], 64, 50, 15, 16) == G.DENSE


# ---------------------------------------------------------------------------
# a4 / a7: normalised aggregation (all widths, both pitches, epilogues)
# ---------------------------------------------------------------------------

WIDTHS = [1, 2, 3, 4, 5, 7, 8, 15, 16, 17, 31, 32, 33, 40, 41, 47, 63, 64, 65, 100, 127, 128, 129,
          256, 257, 602]


@pytest.fixture(scope="module")
def agg_graph(G, orc):
    rng = np.random.default_rng(5)
    s1, d1 = gs.chung_lu(3000, 20000, seed=3)
    s2 = np.zeros(5000, np.int32) + 7
    d2 = rng.integers(0, 3000, 5000).astype(np.int32)     # one hub of degree ~2600
    s = np.concatenate([s1, s2])
    d = np.concatenate([d1, d2])
    return orc.build_csr(3000, s, d), G.build_csr(3000, dev(s), dev(d))


@pytest.mark.parametrize("w", WIDTHS)
@pytest.mark.parametrize("vec", [True, False])
def test_aggregate_widths(G, orc, agg_graph, w, vec):
    og, dg = agg_graph
    rng = np.random.default_rng(w)
    n = og.n
    M = rng.standard_normal((n, w)).astype(np.float32)
    b = rng.standard_normal(w).astype(np.float32)
    ld = G.pitch(w) if vec else w
    Md = pitched(M, ld)
    Zd = pitched(np.zeros((n, w), np.float32), ld)
    mask = rng.standard_normal((n, w)).astype(np.float32)
    Z, mag = orc.aggregate(og, M, b, want_mag=True)
    for epi in (G.EPI_NONE, G.EPI_RELU, G.EPI_MASK):
        G.aggregate(dg, Md, Zd, bias=dev(b), epi=epi, mask=pitched(mask, ld) if epi == G.EPI_MASK else None)
        want = Z if epi == G.EPI_NONE else (np.maximum(Z, 0) if epi == G.EPI_RELU else Z * (mask > 0))
        assert_mag_close(host(Zd), want, mag, f"aggregate w={w} ld={ld} epi={epi}")
    # padding columns were never written
    if ld > w:
        assert torch.isnan(Zd.as_strided((n, ld), (ld, 1))[:, w:]).all()


@pytest.fixture(scope="module")
def dense_rows_graph(G, orc):
    """Mean degree about 90: slices of 16 and 32 lanes take more than 8 entries of an
    average row, so the aggregation keeps 16 neighbour loads in flight per lane."""
    s, d = gs.chung_lu(2000, 90000, seed=4)
    return orc.build_csr(2000, s, d), G.build_csr(2000, dev(s), dev(d))


@pytest.mark.parametrize("w", [33, 40, 47, 64, 65, 100, 128])
def test_aggregate_widths_long_rows(G, orc, dense_rows_graph, w):
    og, dg = dense_rows_graph
    assert og.nnz / og.n > 64
    rng = np.random.default_rng(100 + w)
    n = og.n
    M = rng.standard_normal((n, w)).astype(np.float32)
    b = rng.standard_normal(w).astype(np.float32)
    ld = G.pitch(w)
    Md = pitched(M, ld)
    Zd = pitched(np.zeros((n, w), np.float32), ld)
    mask = rng.standard_normal((n, w)).astype(np.float32)
    Z, mag = orc.aggregate(og, M, b, want_mag=True)
    for epi in (G.EPI_NONE, G.EPI_RELU, G.EPI_MASK):
        G.aggregate(dg, Md, Zd, bias=dev(b), epi=epi, mask=pitched(mask, ld) if epi == G.EPI_MASK else None)
        want = Z if epi == G.EPI_NONE else (np.maximum(Z, 0) if epi == G.EPI_RELU else Z * (mask > 0))
        assert_mag_close(host(Zd), want, mag, f"aggregate long rows w={w} epi={epi}")


def test_aggregate_no_bias_deterministic(G, orc, agg_graph):
    og, dg = agg_graph
    M = np.random.default_rng(0).standard_normal((og.n, 256)).astype(np.float32)
    Md = dev(M)
    a = torch.empty_like(Md)
    b = torch.empty_like(Md)
    G.aggregate(dg, Md, a)
    G.aggregate(dg, Md, b)
    assert torch.equal(a, b)
    Z, mag = orc.aggregate(og, M, want_mag=True)
    assert_mag_close(host(a), Z, mag, "aggregate w=256 no bias")


# ---------------------------------------------------------------------------
# a3 (sparse), a8 (sparse): X_csr W and X_csc Q
# ---------------------------------------------------------------------------


@pytest.mark.parametrize("f,w,p", [(1433, 16, 0.013), (4096, 128, 0.01), (500, 7, 0.2), (300, 33, 0.05)])
def test_sparse_feature_products(G, orc, f, w, p):
    n = 2708
    X = gs.features_bernoulli(n, f, p, seed=1, binary=False)
    rng = np.random.default_rng(f)
    W = rng.standard_normal((f, w)).astype(np.float32)
    Q = rng.standard_normal((n, w)).astype(np.float32)
    _, sx = G.feature_stats(dev(X), materialize=True)
    out = torch.empty((n, w), dtype=torch.float32, device="cuda")
    G.spmm(sx.row_ptr, sx.col[:sx.nnz], sx.val[:sx.nnz], dev(W), out)
    rp, col, val = orc.dense_to_csr(X)
    ref, mag = orc.spmm(rp, col, val, W, want_mag=True)
    assert_mag_close(host(out), ref, mag, f"X_csr W f={f} w={w}")
    dW = torch.empty((f, w), dtype=torch.float32, device="cuda")
    G.spmm(sx.col_ptr, sx.row[:sx.nnz], sx.cval[:sx.nnz], dev(Q), dW)
    cp, row, cval = orc.dense_to_csc(X)
    ref, mag = orc.spmm(cp, row, cval, Q, want_mag=True)
    assert_mag_close(host(dW), ref, mag, f"X_csc Q f={f} w={w}")


# ---------------------------------------------------------------------------
# a3 / a5 / a8 / a9: matrix-core GEMMs
# ---------------------------------------------------------------------------

GEMM_SHAPES = [(1000, 256, 128), (1000, 40, 256), (777, 47, 256), (513, 7, 16), (300, 128, 602),
               (333, 256, 256), (65, 16, 1433), (2049, 41, 41), (1, 1, 1), (100, 300, 5)]


@pytest.mark.parametrize("op", ["NN", "NT", "TN"])
@pytest.mark.parametrize("shape", GEMM_SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_gemm(G, op, shape):
    m, n, k = shape
    rng = np.random.default_rng(m * 7 + n * 3 + k)
    A = rng.standard_normal((m, k)).astype(np.float32)
    B = rng.standard_normal((k, n)).astype(np.float32)
    bias = rng.standard_normal(n).astype(np.float32)
    mask = rng.standard_normal((m, n)).astype(np.float32)
    ref = A.astype(np.float64) @ B.astype(np.float64)
    mag = np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64))
    if op == "NN":
        Ad, Bd, code = pitched(A, G.pitch(k) + 4), pitched(B, G.pitch(n)), G.OP_NN
    elif op == "NT":
        Ad, Bd, code = pitched(A, k), pitched(np.ascontiguousarray(B.T), G.pitch(k)), G.OP_NT
    else:
        Ad, Bd, code = pitched(np.ascontiguousarray(A.T), G.pitch(m)), pitched(B, n), G.OP_TN
    C = pitched(np.zeros((m, n), np.float32), G.pitch(n) + 8)
    G.gemm(code, Ad, Bd, C, bias=dev(bias))
    assert_mag_close(host(C), ref + bias, mag + np.abs(bias), f"gemm {op} {shape}")
    if op != "TN":
        G.gemm(code, Ad, Bd, C, bias=dev(bias), epi=G.EPI_RELU)
        assert_mag_close(host(C), np.maximum(ref + bias, 0), mag + np.abs(bias), f"gemm {op} relu")
        G.gemm(code, Ad, Bd, C, epi=G.EPI_MASK, mask=dev(mask))
        assert_mag_close(host(C), ref * (mask > 0), mag, f"gemm {op} mask")


def test_gemm_huge_pitch(G):
    """Operands whose pitch is too large for 32-bit tile offsets (the fp32-mode fallback)."""
    rng = np.random.default_rng(5)
    m, n, k, ld = 3, 40, 70, (1 << 21) + 4
    A = rng.standard_normal((m, k)).astype(np.float32)
    B = rng.standard_normal((k, n)).astype(np.float32)
    Ad = pitched(A, ld)
    C = torch.empty((m, n), dtype=torch.float32, device="cuda")
    G.gemm(G.OP_NN, Ad, dev(B), C)
    ref = A.astype(np.float64) @ B.astype(np.float64)
    mag = np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64))
    assert_mag_close(host(C), ref, mag, "gemm NN huge pitch")


@pytest.mark.parametrize("m,n,k", [(128, 256, 169343), (256, 40, 50000), (100, 256, 70001), (602, 41, 20000),
                                   (4096, 128, 4000), (16, 7, 2708)])
def test_gemm_tn_long_reduction(G, m, n, k):
    rng = np.random.default_rng(k)
    A = rng.standard_normal((k, m)).astype(np.float32)
    B = rng.standard_normal((k, n)).astype(np.float32)
    ref = A.T.astype(np.float64) @ B.astype(np.float64)
    mag = np.abs(A.T.astype(np.float64)) @ np.abs(B.astype(np.float64))
    C = torch.empty((m, n), dtype=torch.float32, device="cuda")
    G.gemm(G.OP_TN, dev(A), dev(B), C)
    C1 = host(C).copy()
    assert_mag_close(C1, ref, mag, f"gemm TN {m}x{n}x{k}")
    G.gemm(G.OP_TN, dev(A), dev(B), C)
    np.testing.assert_array_equal(host(C), C1)  # fixed-order split-k reduction


# Row-panel products (A B, A B^T with n <= 256, m >= 128, no mask): every column-tile count
# 1..8 (and so every A prefetch depth), partial and single k slabs, ragged row blocks; the
# masked product of the same operands runs on the tiled kernel.
ROWS_CASES = [(256, 1, 5), (1000, 33, 32), (4099, 64, 40), (777, 65, 256), (300, 100, 602), (2048, 130, 64),
              (513, 190, 100), (1500, 220, 17), (1025, 256, 256), (600, 256, 33)]


@pytest.mark.parametrize("op", ["NN", "NT"])
@pytest.mark.parametrize("shape", ROWS_CASES, ids=lambda s: "x".join(map(str, s)))
def test_gemm_row_panels(G, op, shape, monkeypatch):
    monkeypatch.setenv("GCN_GEMM_ROWS", "1")  # below the automatic row threshold
    m, n, k = shape
    rng = np.random.default_rng(m + 3 * n + 7 * k)
    A = (rng.standard_normal((m, k)) * np.exp(rng.standard_normal((m, 1)))).astype(np.float32)
    B = rng.standard_normal((k, n)).astype(np.float32)
    bias = rng.standard_normal(n).astype(np.float32)
    mask = rng.standard_normal((m, n)).astype(np.float32)
    ref = A.astype(np.float64) @ B.astype(np.float64)
    mag = np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64))
    Ad = pitched(A, G.pitch(k))
    Bd = pitched(B, n) if op == "NN" else pitched(np.ascontiguousarray(B.T), k)
    code = G.OP_NN if op == "NN" else G.OP_NT
    C = pitched(np.full((m, n), np.nan, np.float32), G.pitch(n) + 4)
    G.gemm(code, Ad, Bd, C, bias=dev(bias))
    C1 = host(C).copy()
    assert_mag_close(C1, ref + bias, mag + np.abs(bias), f"rows {op} {shape}")
    G.gemm(code, Ad, Bd, C, bias=dev(bias))
    np.testing.assert_array_equal(host(C), C1)  # fixed summation order
    G.gemm(code, Ad, Bd, C, bias=dev(bias), epi=G.EPI_RELU)
    assert_mag_close(host(C), np.maximum(ref + bias, 0), mag + np.abs(bias), f"rows {op} relu")
    G.gemm(code, Ad, Bd, C, epi=G.EPI_MASK, mask=dev(mask))
    assert_mag_close(host(C), ref * (mask > 0), mag, f"rows {op} mask")


@pytest.mark.parametrize("op", ["NN", "NT"])
@pytest.mark.parametrize("shape", [(600, 256, 33), (4099, 250, 40), (300, 226, 64), (1025, 256, 256), (777, 240, 130)],
                         ids=lambda s: "x".join(map(str, s)))
def test_gemm_row_panels_column_groups(G, op, shape, monkeypatch):
    """Few row panels: the 8 column tiles go to two workgroups of 4; every output element keeps
    its summation order, so the result equals the one-group launch bit for bit."""
    monkeypatch.setenv("GCN_GEMM_ROWS", "1")
    m, n, k = shape
    rng = np.random.default_rng(m + n + k)
    A = rng.standard_normal((m, k)).astype(np.float32)
    B = rng.standard_normal((k, n)).astype(np.float32)
    bias = rng.standard_normal(n).astype(np.float32)
    Ad = pitched(A, G.pitch(k))
    Bd = pitched(B, n) if op == "NN" else pitched(np.ascontiguousarray(B.T), k)
    code = G.OP_NN if op == "NN" else G.OP_NT
    out = []
    for groups in ("auto", "1"):
        if groups == "1":
            monkeypatch.setenv("GCN_ROWS_GROUPS", "1")
        C = pitched(np.full((m, n), np.nan, np.float32), G.pitch(n))
        G.gemm(code, Ad, Bd, C, bias=dev(bias), epi=G.EPI_RELU)
        out.append(host(C).copy())
    ref = np.maximum(A.astype(np.float64) @ B.astype(np.float64) + bias, 0)
    mag = np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64)) + np.abs(bias)
    assert_mag_close(out[0], ref, mag, f"column groups {op} {shape}")
    np.testing.assert_array_equal(out[0], out[1])


@pytest.mark.parametrize("op,n,k,epi", [("NN", 256, 256, "none"), ("NT", 256, 256, "mask"), ("NN", 40, 256, "none"),
                                        ("NT", 256, 40, "mask"), ("NN", 256, 128, "relu")])
def test_gemm_row_panels_full_size(G, op, n, k, epi):
    """The transform and input-gradient products at the arxiv-like layer sizes (169,343 rows),
    checked on sampled rows against fp64."""
    m = 169343
    rng = np.random.default_rng(n + k)
    A = dev(rng.standard_normal((m, k), dtype=np.float32))
    B = rng.standard_normal((k, n)).astype(np.float32)
    mask = dev(rng.standard_normal((m, n), dtype=np.float32)) if epi == "mask" else None
    Bd = dev(B) if op == "NN" else dev(np.ascontiguousarray(B.T))
    C = torch.empty((m, n), dtype=torch.float32, device="cuda")
    code = {"none": G.EPI_NONE, "mask": G.EPI_MASK, "relu": G.EPI_RELU}[epi]
    G.gemm(G.OP_NN if op == "NN" else G.OP_NT, A, Bd, C, epi=code, mask=mask)
    rows = np.unique(np.concatenate([rng.integers(0, m, 2000), [0, 255, 256, m - 1]]))
    As = host(A[rows]).astype(np.float64)
    ref = As @ B.astype(np.float64)
    mag = np.abs(As) @ np.abs(B.astype(np.float64))
    if epi == "mask":
        ref = ref * (host(mask[rows]) > 0)
    if epi == "relu":
        ref = np.maximum(ref, 0)
    assert_mag_close(host(C[rows]), ref, mag, f"rows {op} full size {n}x{k}")


@pytest.mark.parametrize("m,n,k", [(1, 1, 17), (33, 40, 1000), (256, 256, 5000), (100, 256, 70001),
                                   (256, 40, 50000), (200, 7, 33333), (64, 256, 123), (160, 96, 65)])
def test_gemm_tn_ragged(G, m, n, k):
    """A^T B on ragged output tiles, partial k slabs and split-k ranges (with a bias)."""
    rng = np.random.default_rng(m * 31 + n + k)
    A = (rng.standard_normal((k, m)) * np.exp(rng.standard_normal((k, 1)))).astype(np.float32)
    B = rng.standard_normal((k, n)).astype(np.float32)
    bias = rng.standard_normal(n).astype(np.float32)
    ref = A.T.astype(np.float64) @ B.astype(np.float64) + bias
    mag = np.abs(A.T.astype(np.float64)) @ np.abs(B.astype(np.float64)) + np.abs(bias)
    Ad, Bd = pitched(A, G.pitch(m) + 4), pitched(B, G.pitch(n))
    C = pitched(np.full((m, n), np.nan, np.float32), G.pitch(n))
    G.gemm(G.OP_TN, Ad, Bd, C, bias=dev(bias))
    C1 = host(C).copy()
    assert_mag_close(C1, ref, mag, f"TN ragged {m}x{n}x{k}")
    G.gemm(G.OP_TN, Ad, Bd, C, bias=dev(bias))
    np.testing.assert_array_equal(host(C), C1)  # fixed-order reduction


# ---------------------------------------------------------------------------
# bias gradient / loss mean, Adam
# ---------------------------------------------------------------------------


@pytest.mark.parametrize("rows,w", [(169343, 256), (2708, 7), (1000, 300), (8192, 40), (8193, 40), (5, 1),
                                    (0, 3)])
@pytest.mark.parametrize("with_rv", [True, False])
def test_column_sums(G, rows, w, with_rv):
    """Column sums with and without the per-row values' mean (the loss pass's form and the
    plain bias gradient share one summation order)."""
    rng = np.random.default_rng(rows + w)
    Gm = rng.standard_normal((rows, w)).astype(np.float32)
    rv = rng.random(rows).astype(np.float32)
    out = torch.full((max(w, 1),), float("nan"), dtype=torch.float32, device="cuda")
    mean = torch.empty(1, dtype=torch.float32, device="cuda")
    use_rv = with_rv and rows > 0
    G.column_sums(pitched(Gm, G.pitch(w)), out[:w], row_vals=dev(rv) if use_rv else None,
                  mean=mean if use_rv else None)
    want = Gm.astype(np.float64).sum(0)
    mag = np.abs(Gm.astype(np.float64)).sum(0)
    assert_mag_close(host(out)[:w], want, mag, "column sums")
    if use_rv:
        assert host(mean)[0] == pytest.approx(rv.astype(np.float64).mean(), rel=1e-6)
    # fixed summation order: a second call gives the same bits
    again = torch.empty_like(out)
    G.column_sums(pitched(Gm, G.pitch(w)), again[:w], row_vals=dev(rv) if use_rv else None,
                  mean=torch.empty_like(mean) if use_rv else None)
    assert torch.equal(out[:w], again[:w])


def test_adam(G, orc):
    rng = np.random.default_rng(3)
    shapes = [(128, 256), (256,), (256, 40), (40,), (7,)]
    ps = [rng.standard_normal(s).astype(np.float32) for s in shapes]
    gs_ = [rng.standard_normal(s).astype(np.float32) for s in shapes]
    ms = [rng.standard_normal(s).astype(np.float32) * 0.1 for s in shapes]
    vs = [rng.random(s).astype(np.float32) * 0.01 for s in shapes]
    dp, dg, dm, dv = ([dev(a) for a in arrs] for arrs in (ps, gs_, ms, vs))
    G.adam(dp, dg, dm, dv, step=3)
    for i in range(len(shapes)):
        want, wm, wv = orc.adam(ps[i], gs_[i], ms[i], vs[i], 3)
        np.testing.assert_allclose(host(dm[i]), wm, rtol=2e-6, atol=1e-7)
        np.testing.assert_allclose(host(dv[i]), wv, rtol=2e-6, atol=1e-9)
        assert_mag_close(host(dp[i]), want, np.abs(ps[i]) + 0.01, f"adam tensor {i}", rtol=1e-5)


# ---------------------------------------------------------------------------
# hub rows split into chunks (rows longer than GCN_SPLIT_MIN entries)
# ---------------------------------------------------------------------------


def expected_plan(ptr, chunk, minlen):
    lens = np.diff(ptr)
    rows = np.nonzero(lens > minlen)[0]
    nch = (lens[rows] + chunk - 1) // chunk
    first = np.concatenate([[0], np.cumsum(nch)])
    owner = np.repeat(np.arange(rows.size), nch)
    return rows, first, owner


@pytest.fixture(scope="module")
def hub_graph(G, orc):
    rng = np.random.default_rng(9)
    n = 20000
    s1, d1 = gs.chung_lu(n, 60000, seed=5)
    hubs = [(3, 15000), (11, 5000), (12, 4000), (19999, 4200)]
    ss, dd = [s1], [d1]
    for h, k in hubs:
        ss.append(np.full(k, h, np.int32))
        dd.append(rng.choice(n, k, replace=False).astype(np.int32))
    s = np.concatenate(ss)
    d = np.concatenate(dd)
    og = orc.build_csr(n, s, d)
    dg = G.build_csr(n, dev(s), dev(d))
    rows, first, owner = expected_plan(og.row_ptr, G.SPLIT_CHUNK, G.SPLIT_MIN)
    assert dg.n_long == rows.size >= 3
    assert dg.c.split.n_chunk == first[-1]
    np.testing.assert_array_equal(host(dg.plan.rows)[:rows.size], rows)
    np.testing.assert_array_equal(host(dg.plan.first)[:rows.size + 1], first)
    np.testing.assert_array_equal(host(dg.plan.owner)[:first[-1]], owner)
    return og, dg


@pytest.mark.parametrize("w", [7, 40, 128, 256])
def test_aggregate_split_hubs(G, orc, hub_graph, w):
    og, dg = hub_graph
    rng = np.random.default_rng(w + 1)
    n = og.n
    M = rng.standard_normal((n, w)).astype(np.float32)
    b = rng.standard_normal(w).astype(np.float32)
    mask = rng.standard_normal((n, w)).astype(np.float32)
    ld = G.pitch(w)
    Md = pitched(M, ld)
    Zd = pitched(np.zeros((n, w), np.float32), ld)
    Z, mag = orc.aggregate(og, M, b, want_mag=True)
    for epi in (G.EPI_NONE, G.EPI_RELU, G.EPI_MASK):
        G.aggregate(dg, Md, Zd, bias=dev(b), epi=epi, mask=pitched(mask, ld) if epi == G.EPI_MASK else None)
        want = Z if epi == G.EPI_NONE else (np.maximum(Z, 0) if epi == G.EPI_RELU else Z * (mask > 0))
        assert_mag_close(host(Zd), want, mag, f"split aggregate w={w} epi={epi}")
    first = host(Zd).copy()
    G.aggregate(dg, Md, Zd, bias=dev(b), epi=G.EPI_MASK, mask=pitched(mask, ld))
    np.testing.assert_array_equal(host(Zd), first)


def test_softmax_layer_on_split_hubs(G, orc, hub_graph):
    og, dg = hub_graph
    n = og.n
    rng = np.random.default_rng(4)
    H = np.maximum(rng.standard_normal((n, 64)), 0).astype(np.float32)
    W = (rng.standard_normal((64, 41)) / 8).astype(np.float32)
    b = (rng.standard_normal(41) * 0.1).astype(np.float32)
    y = rng.integers(0, 41, n).astype(np.int32)
    L = G.make_layer(64, 41, 64, G.pitch(41), G.ACT_SOFTMAX_CE, 1)
    Hd = pitched(H, 64)
    out = pitched(np.zeros((n, 41), np.float32), G.pitch(41))
    logits = pitched(np.zeros((n, 41), np.float32), G.pitch(41))
    loss = torch.zeros(1, device="cuda")
    G.layer_fwd(dg, L, Hd, None, dev(W), dev(b), out, labels=dev(y), loss=loss, logits=logits)
    Z = orc.aggregate(og, orc.matmul(H, W), b)
    mag = orc.aggregate(og, orc.matmul(np.abs(H), np.abs(W)), np.abs(b))
    assert_mag_close(host(logits), Z, mag, "split logits")
    lo, Gr, _ = orc.softmax_ce(Z, y)
    assert host(loss)[0] == pytest.approx(lo, rel=1e-4)
    np.testing.assert_allclose(host(out), Gr, rtol=0, atol=1e-4 * np.abs(Gr).max())


def length_class(d):
    """Processing class of a row of length d (0 first): 4 classes per power of two of d."""
    d = np.asarray(d, np.int64)
    lg = np.floor(np.log2(np.maximum(d, 1))).astype(np.int64)
    key = np.where(d < 4, d, 4 * lg + ((d >> np.maximum(lg - 2, 0)) & 3))
    return np.where(d < 4, 63 - d, 63 - np.minimum(key, 63))


@pytest.mark.parametrize("case", ["hubs", "dense", "cora_like", "empty"])
def test_row_order(G, orc, hub_graph, case):
    """The row order of the aggregations: a permutation of the rows, by length class, longest
    first, ties in row order; and every aggregation result (all epilogues, split hub rows,
    the loss epilogue) is bit-identical with and without it.  The order is applied where an
    average row gathers at least 4 KB: on the dense graph (about 67 entries per row) at every
    width here, on the others at width 256."""
    if case == "hubs":
        og, dg = hub_graph
        s = d = None
    elif case == "dense":
        s, d = gs.chung_lu(6000, 200000, seed=8)
        og, dg = orc.build_csr(6000, s, d), G.build_csr(6000, dev(s), dev(d))
        assert og.nnz / og.n * 4 * 7 < 4096 < og.nnz / og.n * 4 * 40
    elif case == "cora_like":
        wl = gs.WORKLOADS["cora_like"]
        s, d = gs.make_graph(wl)
        og, dg = orc.build_csr(wl.n, s, d), G.build_csr(wl.n, dev(s), dev(d))
    else:
        s = d = np.zeros(0, np.int32)
        og, dg = orc.build_csr(300, s, d), G.build_csr(300, dev(s), dev(d))
    n = og.n
    order = host(dg.order)[:n]
    np.testing.assert_array_equal(np.sort(order), np.arange(n))
    cls = length_class(og.deg)[order]
    key = cls.astype(np.int64) * (n + 1) + order
    assert np.all(np.diff(key) > 0), "classes ascending (longest first), rows ascending within a class"
    if case == "hubs":
        e = host(dg.row_ptr)
        s_ = np.repeat(np.arange(n, dtype=np.int32), np.diff(e))
        d_ = host(dg.col_idx)[:og.nnz]
    else:
        s_, d_ = s, d
    plain = G.build_csr(n, dev(s_), dev(d_), order=False)
    assert plain.order is None and plain.nnz == dg.nnz
    rng = np.random.default_rng(n)
    for w in (7, 16, 40, 256):
        M = pitched(rng.standard_normal((n, w)).astype(np.float32), G.pitch(w))
        b = dev(rng.standard_normal(w).astype(np.float32))
        mask = pitched(rng.standard_normal((n, w)).astype(np.float32), G.pitch(w))
        for epi in (G.EPI_NONE, G.EPI_RELU, G.EPI_MASK):
            outs = []
            for g in (dg, plain):
                Z = pitched(np.zeros((n, w), np.float32), G.pitch(w))
                G.aggregate(g, M, Z, bias=b, epi=epi, mask=mask if epi == G.EPI_MASK else None)
                outs.append(host(Z))
            np.testing.assert_array_equal(outs[0], outs[1])
    # the loss epilogue (rows taken in groups of slots consecutive positions of the order)
    H = pitched(np.maximum(rng.standard_normal((n, 64)), 0).astype(np.float32), 64)
    W = dev((rng.standard_normal((64, 41)) / 8).astype(np.float32))
    bb = dev((rng.standard_normal(41) * 0.1).astype(np.float32))
    y = dev(rng.integers(0, 41, n).astype(np.int32))
    L = G.make_layer(64, 41, 64, G.pitch(41), G.ACT_SOFTMAX_CE, 1)
    res = []
    for g in (dg, plain):
        out = pitched(np.zeros((n, 41), np.float32), G.pitch(41))
        logits = pitched(np.zeros((n, 41), np.float32), G.pitch(41))
        loss = torch.zeros(1, device="cuda")
        G.layer_fwd(g, L, H, None, W, bb, out, labels=y, loss=loss, logits=logits)
        res.append((host(out), host(logits), host(loss)))
    for a, c in zip(*res):
        np.testing.assert_array_equal(a, c)


def test_tune_row_order(G, orc):
    """The tuner keeps or drops the order; either way the graph aggregates as before."""
    wl = gs.WORKLOADS["cora_like"]
    s, d = gs.make_graph(wl)
    g = G.build_csr(wl.n, dev(s), dev(d))
    rng = np.random.default_rng(3)
    M = pitched(rng.standard_normal((wl.n, 40)).astype(np.float32), G.pitch(40))
    before = pitched(np.zeros((wl.n, 40), np.float32), G.pitch(40))
    G.aggregate(g, M, before)
    kept = G.tune_row_order(g, 40)
    assert kept == (g.order is not None) and (g.c.order is not None) == kept
    after = pitched(np.zeros((wl.n, 40), np.float32), G.pitch(40))
    G.aggregate(g, M, after)
    np.testing.assert_array_equal(host(after), host(before))


@pytest.mark.parametrize("fi,fo", [(128, 256), (48, 300)])
def test_aggregate_first_layer_on_split_hubs(G, orc, hub_graph, fi, fo):
    """Aggregate-then-transform layer: hub rows come from the chunk sums."""
    og, dg = hub_graph
    n = og.n
    rng = np.random.default_rng(fi)
    H = rng.standard_normal((n, fi)).astype(np.float32)
    W = (rng.standard_normal((fi, fo)) / np.sqrt(fi)).astype(np.float32)
    b = (rng.standard_normal(fo) * 0.1).astype(np.float32)
    L = G.make_layer(fi, fo, G.pitch(fi), G.pitch(fo), G.ACT_RELU, 0, G.AGGREGATE_FIRST)
    out = pitched(np.zeros((n, fo), np.float32), G.pitch(fo))
    saved = pitched(np.zeros((n, fi), np.float32), G.pitch(fi))
    G.layer_fwd(dg, L, pitched(H, G.pitch(fi)), None, dev(W), dev(b), out, saved=saved)
    P, pmag = orc.aggregate(og, H, want_mag=True)
    assert_mag_close(host(saved), P, pmag, "split hubs: saved A_hat H")
    Z = orc.aggregate(og, orc.matmul(H, W), b)
    mag = orc.aggregate(og, orc.matmul(np.abs(H), np.abs(W)), np.abs(b))
    assert_mag_close(host(out), np.maximum(Z, 0), mag, f"split hubs: AF {fi}->{fo}")


# ---------------------------------------------------------------------------
# other aggregators: sum, mean and its transpose, max (forward and gradient)
# ---------------------------------------------------------------------------

AGG_CODE = {"sum": 1, "mean": 2, "mean_t": 3}


@pytest.mark.parametrize("kind", ["sum", "mean", "mean_t"])
@pytest.mark.parametrize("w", [7, 40, 256])
def test_linear_aggregators_on_split_hubs(G, orc, hub_graph, kind, w):
    og, dg = hub_graph
    rng = np.random.default_rng(w + 7)
    n = og.n
    M = rng.standard_normal((n, w)).astype(np.float32)
    b = rng.standard_normal(w).astype(np.float32)
    mask = rng.standard_normal((n, w)).astype(np.float32)
    ld = G.pitch(w)
    Md = pitched(M, ld)
    Zd = pitched(np.zeros((n, w), np.float32), ld)
    Z, mag = orc.aggregate(og, M, b, want_mag=True, kind=kind)
    for epi in (G.EPI_NONE, G.EPI_RELU, G.EPI_MASK):
        G.aggregate(dg, Md, Zd, bias=dev(b), epi=epi, mask=pitched(mask, ld) if epi == G.EPI_MASK else None,
                    agg=AGG_CODE[kind])
        want = Z if epi == G.EPI_NONE else (np.maximum(Z, 0) if epi == G.EPI_RELU else Z * (mask > 0))
        assert_mag_close(host(Zd), want, mag, f"{kind} aggregate w={w} epi={epi}")


@pytest.mark.parametrize("w,ld", [(7, 7), (7, 8), (40, 40), (128, 128), (256, 256), (41, 41)])
def test_max_aggregation_bit_exact_with_ties(G, orc, hub_graph, w, ld):
    """Max and first maximiser are exact in fp32: equal to the oracle bit for bit, also on
    rows of small integers (many ties) and on the hub rows (walked by one lane group)."""
    og, dg = hub_graph
    n = og.n
    rng = np.random.default_rng(w * 3 + ld)
    M = rng.integers(-3, 4, (n, w)).astype(np.float32)
    M[::7] = rng.standard_normal((M[::7].shape)).astype(np.float32)
    Pd = pitched(np.zeros((n, w), np.float32), ld)
    argd = torch.zeros((n, ld), dtype=torch.int32, device="cuda")[:, :w]
    G.aggregate_max(dg, pitched(M, ld), Pd, argd)
    P, arg = orc.aggregate_max(og, M)
    np.testing.assert_array_equal(host(Pd), P.astype(np.float32))
    np.testing.assert_array_equal(host(argd), arg)
    # gradient: the gather over the symmetric rows against the oracle's scatter
    dP = rng.standard_normal((n, w)).astype(np.float32)
    mask = rng.standard_normal((n, w)).astype(np.float32)
    dMd = pitched(np.zeros((n, w), np.float32), ld)
    for use_mask in (False, True):
        G.aggregate_max_bwd(dg, pitched(dP, ld), argd, dMd, mask=pitched(mask, ld) if use_mask else None)
        want = orc.aggregate_max_backward(og, dP, arg)
        mag = orc.aggregate_max_backward(og, np.abs(dP), arg)
        if use_mask:
            want, mag = want * (mask > 0), mag * (mask > 0)
        assert_mag_close(host(dMd), want, mag, f"max gradient w={w} mask={use_mask}")
    first = host(dMd).copy()
    G.aggregate_max_bwd(dg, pitched(dP, ld), argd, dMd, mask=pitched(mask, ld))
    np.testing.assert_array_equal(host(dMd), first)  # fixed order


def test_sparse_backward_atomic_transpose(G, orc):
    """X^T Q from the CSR rows with atomic adds (no CSC view): within the fp32 bar of the
    oracle; the rounding order may differ between runs, the values stay within it."""
    n, f, w = 20000, 300, 40
    X = gs.features_bernoulli(n, f, 0.05, seed=4, binary=False)
    rng = np.random.default_rng(3)
    Q = rng.standard_normal((n, w)).astype(np.float32)
    info, sx = G.feature_stats(dev(X), force_mode=G.SPARSE, csc=False)
    assert sx.col_ptr is None
    L = G.make_layer(f, w, f, G.pitch(w), G.ACT_RELU, 0)
    dW = torch.zeros((f, w), device="cuda")
    db = torch.zeros(w, device="cuda")
    g = G.build_csr(n, dev(np.zeros(0, np.int32)), dev(np.zeros(0, np.int32)))  # A + I = I: Q passes through
    G.layer_bwd(g, L, pitched(Q, G.pitch(w)), None, sx, None, dev(np.zeros((f, w), np.float32)), dW, db, None)
    rp, col, val = orc.dense_to_csr(X)
    want = orc.matmul(X.T, Q)
    mag = orc.matmul(np.abs(X).T, np.abs(Q))
    assert_mag_close(host(dW), want, mag, "atomic X^T Q")


def test_sparse_backward_long_columns(G, orc):
    """X with few, dense columns: every CSC column is long and goes through chunks
    processed chunk-index-major."""
    n, f, w = 30000, 48, 40
    X = gs.features_bernoulli(n, f, 0.4, seed=2, binary=False)
    rng = np.random.default_rng(1)
    Q = rng.standard_normal((n, w)).astype(np.float32)
    _, sx = G.feature_stats(dev(X), materialize=True)
    cp, row, cval = orc.dense_to_csc(X)
    rows, first, owner = expected_plan(cp, G.SPLIT_CHUNK, G.SPLIT_MIN)
    sp = sx.c.csc_split
    assert sp.n_long == rows.size == f and sp.n_chunk == first[-1]
    np.testing.assert_array_equal(host(sx.plan.first)[:f + 1], first)
    order = host(sx.plan.order)[:first[-1]]
    np.testing.assert_array_equal(np.sort(order), np.arange(first[-1]))
    k_of = order - first[owner[order]]
    assert (np.diff(k_of) >= 0).all()          # chunk index never decreases along the order
    dW = torch.empty((f, w), dtype=torch.float32, device="cuda")
    G.spmm(sx.col_ptr, sx.row[:sx.nnz], sx.cval[:sx.nnz], dev(Q), dW, split=sp)
    ref, mag = orc.spmm(cp, row, cval, Q, want_mag=True)
    assert_mag_close(host(dW), ref, mag, "X_csc Q with long columns")


@pytest.mark.parametrize("op", ["NN", "NT", "TN"])
@pytest.mark.parametrize("shape", [(4000, 256, 256), (3000, 40, 602), (777, 128, 4096), (50000, 64, 100)],
                         ids=lambda s: "x".join(map(str, s)))
def test_gemm_bf16x6_matches_native_fp32(G, op, shape, monkeypatch):
    """The bf16x6 split (default) and native fp32 MFMA agree to fp32 accuracy."""
    m, n, k = shape
    rng = np.random.default_rng(m + n + k)
    A = (rng.standard_normal((m, k)) * np.exp(rng.standard_normal((m, 1)))).astype(np.float32)
    B = rng.standard_normal((k, n)).astype(np.float32)
    if op == "NN":
        Ad, Bd, code = dev(A), dev(B), G.OP_NN
    elif op == "NT":
        Ad, Bd, code = dev(A), dev(np.ascontiguousarray(B.T)), G.OP_NT
    else:
        Ad, Bd, code = dev(np.ascontiguousarray(A.T)), dev(B), G.OP_TN
    mag = np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64))
    ref = A.astype(np.float64) @ B.astype(np.float64)
    out = {}
    for mode in ("bf16x6", "fp32"):
        monkeypatch.setenv("GCN_GEMM_MODE", mode)
        C = torch.empty((m, n), dtype=torch.float32, device="cuda")
        G.gemm(code, Ad, Bd, C)
        out[mode] = host(C).astype(np.float64)
        assert_mag_close(out[mode], ref, mag, f"{mode} {op} {shape}")
    worst = assert_mag_close(out["bf16x6"], out["fp32"], mag, f"bf16x6 vs fp32 {op} {shape}", rtol=2e-6)
    print(f"bf16x6 vs fp32 {op} {shape}: max |diff| / scale = {worst:.2e}")


@pytest.mark.parametrize("n,e,blocked", [(40000, 4500000, True), (30000, 1100000, False), (30000, 450000, False), (30000, 200000, False), (70, 400, False)])
def test_wide_row_panels(G, orc, n, e, blocked):
    """The panelled aggregation at the edges of its panels (32, 64 and 128 columns; pitches that
    are and are not multiples of a line), for every weight kind and epilogue, unblocked and
    blocked by source rows (two blocks of 24,576 or four of 12,288, and at least 8 M entries),
    rows cut over four wavefronts (more than 512 entries) and, by the split plan, over chunks (more
    than 4,096, or as many per block).  Tolerance: fp32 rounding relative to the sum of
    |terms| of an element, as everywhere here.  The same sums come out bit for bit again and
    without the row order."""
    s, d = gs.chung_lu(n, e, seed=3, dmax=min(n // 4, 6000.0))
    og, dg = orc.build_csr(n, s, d), G.build_csr(n, dev(s), dev(d))
    plain = G.build_csr(n, dev(s), dev(d), order=False)
    if n > 1000:
        assert og.deg.max() > 512
    if blocked:
        assert og.nnz >= 8_000_000 and dg.n_long > 0
    rng = np.random.default_rng(e)
    rows = np.unique(np.concatenate([rng.integers(0, n, 200), np.argsort(og.deg)[-20:], np.argsort(og.deg)[:20]]))
    M = rng.standard_normal((n, 260)).astype(np.float32)
    bias = rng.standard_normal(260).astype(np.float32)
    mask = rng.standard_normal((n, 260)).astype(np.float32)
    kinds = {"norm": G.AGG_NORM, "sum": G.AGG_SUM, "mean": G.AGG_MEAN, "mean_t": G.AGG_MEAN_T}
    for w, ld in ((1, 4), (5, 8), (16, 16), (17, 20), (32, 32), (33, 48), (64, 64), (65, 68), (100, 100), (128, 128), (129, 132), (256, 256),
                  (260, 288)):
        for kind, epi in (("norm", G.EPI_NONE), ("norm", G.EPI_RELU), ("sum", G.EPI_MASK), ("mean", G.EPI_RELU),
                          ("mean_t", G.EPI_NONE)):
            Md, Kd = pitched(M[:, :w], ld), pitched(mask[:, :w], ld)
            outs = []
            for g in (dg, dg, plain):
                Z = pitched(np.full((n, w), np.nan, np.float32), ld)
                G.aggregate(g, Md, Z, bias=dev(bias[:w]), epi=epi, mask=Kd if epi == G.EPI_MASK else None,
                            agg=kinds[kind])
                outs.append(host(Z))
            np.testing.assert_array_equal(outs[0], outs[1])
            np.testing.assert_array_equal(outs[0], outs[2])
            want, mag = orc.aggregate(og, M[:, :w], bias[:w], rows=rows, want_mag=True, kind="gcn" if kind == "norm" else kind)
            if epi == G.EPI_RELU:
                want = np.maximum(want, 0)
            elif epi == G.EPI_MASK:
                want = want * (mask[rows, :w] > 0)
            assert_mag_close(outs[0][rows], want, mag, f"{kind} epi {epi} width {w} pitch {ld}")
    # an infinity reaches exactly the rows that gather it
    Mi = M[:, :64].copy()
    Mi[7, 3] = np.inf
    Z = pitched(np.zeros((n, 64), np.float32), 64)
    G.aggregate(dg, pitched(Mi, 64), Z)
    hit = np.zeros(n, bool)
    hit[np.repeat(np.arange(n), og.deg)[og.col_idx == 7]] = True
    got = host(Z)
    np.testing.assert_array_equal(np.isinf(got[:, 3]), hit)
    assert np.isfinite(np.delete(got, 3, axis=1)).all() and not np.isnan(got).any()


@pytest.mark.parametrize("agg", ["gcn", "mean"])
@pytest.mark.parametrize("w", [7, 24, 33, 41, 64, 100, 128, 129, 256])
def test_loss_epilogue_row_panels(G, orc, w, agg):
    """The loss epilogue over sums that come from several blocks of source rows (33 columns and
    more here), in slices of 16 and 32 lanes that each keep a row of their own, and over several
    panels (64 columns and more than 128).  W is a cut of the identity, so the aggregated matrix is
    the input's first columns.  Logits of every row relative to the sum of |terms|, the gradient
    relative to its largest element, 1e-4 as everywhere here."""
    n, f = 40000, 260
    s, d = gs.chung_lu(n, 4500000, seed=5, dmax=6000.0)
    og, dg = orc.build_csr(n, s, d), G.build_csr(n, dev(s), dev(d))
    assert og.nnz >= 8_000_000
    rng = np.random.default_rng(w)
    H = rng.standard_normal((n, f)).astype(np.float32)
    b = rng.standard_normal(w).astype(np.float32)
    y = rng.integers(0, w, n).astype(np.int32)
    kind = G.AGG_NORM if agg == "gcn" else G.AGG_MEAN
    L = G.make_layer(f, w, f, G.pitch(w), G.ACT_SOFTMAX_CE, 1, agg=kind)
    Hout, logits, loss = G.padded(n, w), G.padded(n, w), torch.zeros(1, device="cuda")
    G.layer_fwd(dg, L, dev(H), None, dev(np.eye(f, w, dtype=np.float32)), dev(b), Hout, labels=dev(y), loss=loss,
                logits=logits)
    Z, mag = orc.aggregate(og, H[:, :w], b, want_mag=True, kind=agg)
    assert_mag_close(host(logits), Z, mag, f"{agg} logits {w}")
    want, Gl, _ = orc.softmax_ce(Z, y)
    assert float(host(loss)[0]) == pytest.approx(want, rel=1e-4)
    assert_norm_close(host(Hout), Gl, f"{agg} loss gradient {w}")


@pytest.mark.parametrize("f,ld", [(1, 1), (31, 32), (33, 33), (128, 128), (257, 260), (1025, 1028), (4097, 4097),
                                  (8200, 8200)])
def test_feature_views_edges(G, orc, f, ld):
    """Counts and both views, byte for byte, at the edges of the words (32 columns), of a
    wavefront's turn (256 to 1,024 columns), of the column blocks (4,096) and of the row chunks
    (64), sparse and dense rows (the views' two forms meet at one nonzero in 20), with rows of
    more than 64 nonzeros, empty rows and columns, NaN, infinities and -0.0, and NaN in the
    padding."""
    rng = np.random.default_rng(f)
    for n, p in ((1, 0.5), (64, 0.0), (65, 0.02), (130, 0.045), (200, 0.055), (63, 1.0)):
        X = np.where(rng.random((n, f)) < p, rng.standard_normal((n, f)), 0.0).astype(np.float32)
        X[n // 2, f // 2] = np.nan
        X[0, f - 1] = -np.inf
        X[n - 1, 0] = -0.0
        Xd = pitched(X, ld)  # NaN in the padding
        info, sx = G.feature_stats(Xd, materialize=True)
        nnz = int((X != 0).sum())
        assert info["nnz"] == nnz and sx.nnz == nnz
        rp, col, val = orc.dense_to_csr(X)
        cp, row, cval = orc.dense_to_csc(X)
        np.testing.assert_array_equal(host(sx.row_ptr), rp)
        np.testing.assert_array_equal(host(sx.col)[:nnz], col)
        np.testing.assert_array_equal(host(sx.val)[:nnz].view(np.int32), val.astype(np.float32).view(np.int32))
        np.testing.assert_array_equal(host(sx.col_ptr), cp)
        np.testing.assert_array_equal(host(sx.row)[:nnz], row)
        np.testing.assert_array_equal(host(sx.cval)[:nnz].view(np.int32), cval.astype(np.float32).view(np.int32))


@pytest.mark.parametrize("n", [1, 2, 1023, 1025, 40000, 600000])
def test_build_csr_row_lengths(G, orc, n):
    """The graph build at the lengths where a row changes hands (64, 128, 256 and 512 raw entries
    sorted by a wavefront, 4,096 by a workgroup, more by the windowed bitmap, one and two windows
    of 2^19 columns), with rows that are all duplicates, duplicates that cross those lengths,
    self pairs, buckets that are split and buckets that are not, and sub-buckets too large for
    LDS: byte for byte the oracle's graph."""
    rng = np.random.default_rng(n)
    src, dst = [np.zeros(0, np.int64)], [np.zeros(0, np.int64)]
    for i, want in enumerate((62, 63, 64, 127, 128, 255, 256, 257, 511, 512, 513, 4094, 4095, 4096, 9000)):
        if i >= n:
            break
        hub = (i * 7919) % n
        src.append(np.full(want, hub))
        dst.append(rng.integers(0, n, want))
    src.append(rng.integers(0, n, 3 * n))
    dst.append(rng.integers(0, n, 3 * n))
    src.append(np.full(700, n // 2))  # one pair, 700 times
    dst.append(np.full(700, n - 1))
    if n >= 40000:
        src.append(np.full(30000, 5))  # a sub-bucket that does not fit, its hub beyond 4,096
        dst.append(rng.permutation(n)[:30000])
    s = np.concatenate(src).astype(np.int32)
    d = np.concatenate(dst).astype(np.int32)
    mix = rng.permutation(s.size)
    s, d = s[mix], d[mix]
    print(f"[build] n {n} pairs {s.size}", flush=True)
    og = orc.build_csr(n, s, d)
    for _ in range(2):
        check_graph_equal(G.build_csr(n, dev(s), dev(d)), og, n)
    # an endpoint out of range is refused wherever it stands
    for bad in (-1, n):
        d2 = d.copy()
        d2[d2.size // 3] = bad
        with pytest.raises(G.GcnError) as e:
            G.build_csr(n, dev(s), dev(d2))
        assert e.value.status == G.E_RANGE


@pytest.mark.parametrize("w,ld", [(17, 20), (33, 36), (64, 64), (100, 100), (128, 128), (256, 256)])
def test_max_row_panels(G, orc, w, ld):
    """The max aggregation and its gradient one row per wavefront, at the edges of the panels, with
    rows cut over four wavefronts, ties (small integers: the first maximiser of many), rows of
    -inf and infinities: maxima and maximisers bit for bit, the gradient to fp32 rounding of its
    sum of |terms|, masked and not."""
    n = 6000
    s, d = gs.chung_lu(n, 60000, seed=5, dmax=2500.0)
    og, dg = orc.build_csr(n, s, d), G.build_csr(n, dev(s), dev(d))
    assert og.deg.max() > 1024
    rng = np.random.default_rng(w)
    M = rng.integers(-3, 4, (n, w)).astype(np.float32)
    M[:, 1] = -np.inf
    M[17, 2] = np.inf
    M[:, 3] = rng.standard_normal(n)
    P, arg = orc.aggregate_max(og, M)
    Pd = pitched(np.zeros((n, w), np.float32), ld)
    argd = torch.full((n, ld), -7, dtype=torch.int32, device="cuda")[:, :w]
    G.aggregate_max(dg, pitched(M, ld), Pd, argd)
    np.testing.assert_array_equal(host(Pd), P.astype(np.float32))
    np.testing.assert_array_equal(host(argd), arg)
    dP = rng.standard_normal((n, w)).astype(np.float32)
    mask = rng.standard_normal((n, w)).astype(np.float32)
    want = orc.aggregate_max_backward(og, dP, arg)
    mag = orc.aggregate_max_backward(og, np.abs(dP), arg)
    for mk in (None, mask):
        dM = pitched(np.full((n, w), np.nan, np.float32), ld)
        G.aggregate_max_bwd(dg, pitched(dP, ld), argd, dM, mask=None if mk is None else pitched(mk, ld))
        keep = 1.0 if mk is None else (mk > 0)
        assert_mag_close(host(dM), want * keep, mag, f"max gradient width {w}")


def sentinel(a, ld, fill):
    """Device copy of a with row pitch ld; the extra columns hold a finite value."""
    buf = torch.full((a.shape[0], ld), fill, dtype=torch.float32, device="cuda")
    buf[:, :a.shape[1]] = dev(a.astype(np.float32))
    return buf[:, :a.shape[1]]


def padding_of(t, ld):
    return host(t.as_strided((t.shape[0], ld), (ld, 1)))[:, t.shape[1]:]


@pytest.mark.parametrize("w,ld", [(17, 20), (33, 36), (41, 44), (41, 64), (47, 48), (101, 128), (602, 604)])
def test_partial_sums_stay_inside_the_width(G, orc, w, ld):
    """The columns between width and pitch are the caller's, also where a row's sum is built up in
    Z by several launches (two or four blocks of source rows here): a finite value there, and another
    one beside M, are found unchanged."""
    n = 40000
    s, d = gs.chung_lu(n, 4500000, seed=3, dmax=6000.0)
    og, dg = orc.build_csr(n, s, d), G.build_csr(n, dev(s), dev(d))
    rng = np.random.default_rng(w)
    rows = rng.integers(0, n, 100)
    M = rng.standard_normal((n, w)).astype(np.float32)
    for epi in (G.EPI_NONE, G.EPI_RELU, G.EPI_MASK):
        Z = sentinel(np.zeros((n, w)), ld, 12345.0)
        mask = sentinel(np.ones((n, w)), ld, 1.0)
        G.aggregate(dg, sentinel(M, ld, 7.0), Z, epi=epi, mask=mask if epi == G.EPI_MASK else None)
        np.testing.assert_array_equal(padding_of(Z, ld), 12345.0)
        want, mag = orc.aggregate(og, M, rows=rows, want_mag=True)
        assert_mag_close(host(Z)[rows], np.maximum(want, 0) if epi == G.EPI_RELU else want, mag, f"width {w} pitch {ld}")


@pytest.mark.parametrize("n,e", [(40000, 4500000), (30000, 450000)])
@pytest.mark.parametrize("fi,fo,order", [(64, 41, "TF"), (130, 129, "TF"), (130, 101, "TF"), (130, 64, "AF")])
def test_layer_outputs_stay_inside_the_width(G, orc, n, e, fi, fo, order):
    """The same for a layer's outputs: the gradient row of the loss epilogue (one panel and two;
    rows of more than 4,096 entries summed in chunks where the graph is not blocked), its logits,
    and the saved aggregate of an aggregate-first layer."""
    s, d = gs.chung_lu(n, e, seed=5, dmax=7000.0)
    dg = G.build_csr(n, dev(s), dev(d))
    assert dg.n_long > 0
    rng = np.random.default_rng(fo)
    H, W = rng.standard_normal((n, fi)), rng.standard_normal((fi, fo)) / np.sqrt(fi)
    ldi, ldo = (fi + 3) // 4 * 4, (fo + 3) // 4 * 4
    act = G.ACT_SOFTMAX_CE if order == "TF" else G.ACT_RELU
    L = G.make_layer(fi, fo, ldi, ldo, act, 1, G.TRANSFORM_FIRST if order == "TF" else G.AGGREGATE_FIRST)
    out, logits = sentinel(np.zeros((n, fo)), ldo, 12345.0), sentinel(np.zeros((n, fo)), ldo, 12345.0)
    saved = sentinel(np.zeros((n, fi)), ldi, 12345.0)
    G.layer_fwd(dg, L, sentinel(H, ldi, 7.0), None, dev(W.astype(np.float32)), dev(np.zeros(fo, np.float32)), out, saved=saved,
                labels=dev(rng.integers(0, fo, n).astype(np.int32)), loss=torch.zeros(1, device="cuda"), logits=logits)
    for t, ld in ((out, ldo), (logits, ldo), (saved, ldi)):
        np.testing.assert_array_equal(padding_of(t, ld), 12345.0)


@pytest.mark.parametrize("k", [1, 64, 65, 100, 128, 129, 200, 256])
def test_gemm_short_reduction_with_epilogue(G, k):
    """A^T B over up to 256 rows takes the ReLU and mask epilogues (a longer reduction may be split
    over workgroups, which applies the bias only)."""
    rng = np.random.default_rng(k)
    for m, n in ((16, 7), (128, 128), (100, 47)):
        A, B = rng.standard_normal((k, m)).astype(np.float32), rng.standard_normal((k, n)).astype(np.float32)
        bias, mask = rng.standard_normal(n).astype(np.float32), rng.standard_normal((m, n)).astype(np.float32)
        A64, B64 = A.astype(np.float64), B.astype(np.float64)
        Z, mag = A64.T @ B64 + bias, np.abs(A64).T @ np.abs(B64) + np.abs(bias)
        for epi in (G.EPI_NONE, G.EPI_RELU, G.EPI_MASK):
            out = torch.full((m, n), float("nan"), device="cuda")
            G.gemm(G.OP_TN, dev(A), dev(B), out, bias=dev(bias), epi=epi, mask=dev(mask) if epi == G.EPI_MASK else None)
            want = Z if epi == G.EPI_NONE else (np.maximum(Z, 0) if epi == G.EPI_RELU else Z * (mask > 0))
            assert_mag_close(host(out), want, mag, f"TN {m}x{n}x{k} epi {epi}")


def test_build_csr_all_pairs_in_one_sub_bucket(G):
    """The largest input there is, 2^30 - 1 pairs, all of the nodes 0 and 1, which share a sub-bucket
    of the partition: 2^31 raw entries there, one more than 31 bits count."""
    n, e = 700000, (1 << 30) - 1
    s, d = torch.zeros(e, dtype=torch.int32, device="cuda"), torch.ones(e, dtype=torch.int32, device="cuda")
    s[::3], d[::3] = 1, 0
    L, g = G.raw_lib(), G.build_csr(n, s[:1], d[:1])
    need = G.sz(0)
    assert L.gcn_build_csr(n, e, None, None, None, None, C.byref(need), None) == G.OK
    ws = torch.empty(need.value, dtype=torch.uint8, device="cuda")
    g.row_ptr.fill_(-1)
    note("2^30 - 1 pairs of two nodes")
    rc = L.gcn_build_csr(n, e, s.data_ptr(), d.data_ptr(), C.byref(g.c), ws.data_ptr(), C.byref(need), None)
    assert rc == G.OK, L.gcn_last_error()
    note("built")
    assert g.c.nnz == n + 2 and host(g.col_idx)[:5].tolist() == [0, 1, 0, 1, 2]
    assert host(g.row_ptr[:4]).tolist() == [0, 2, 4, 5] and int(g.row_ptr[n]) == n + 2
    want = np.float32(1 / np.sqrt(2))
    np.testing.assert_array_equal(host(g.val)[:5], np.array([want * want] * 4 + [1.0], np.float32))


def call_sized(G, fn, before, st, nbytes):
    buf = torch.full((max(nbytes, 256),), 0xEE, dtype=torch.uint8, device="cuda")
    rc = fn(*before, buf.data_ptr(), C.byref(G.sz(nbytes)), st)
    torch.cuda.synchronize()
    return rc


@pytest.mark.parametrize("split", [True, False])
def test_aggregate_with_the_chunk_sums_alone(G, orc, split):
    """gcn_aggregate takes a workspace that holds the chunk sums of the split rows and no more: the
    sums of a dense graph are then not blocked by source rows.  One byte less is refused."""
    n, w = 40000, 64
    s, d = gs.chung_lu(n, 4500000, seed=3, dmax=6000.0)
    og, dg = orc.build_csr(n, s, d), G.build_csr(n, dev(s), dev(d), split=split)
    assert (dg.n_long > 0) == split
    rng = np.random.default_rng(1)
    M = rng.standard_normal((n, w)).astype(np.float32)
    Md, Z = dev(M), torch.full((n, w), float("nan"), device="cuda")
    L, st = G.raw_lib(), C.c_void_p(torch.cuda.current_stream().cuda_stream)
    before = (C.byref(dg.c), G.AGG_NORM, w, Md.data_ptr(), w, None, G.EPI_NONE, None, 0, Z.data_ptr(), w)
    least = 4 * w * dg.c.split.n_chunk if split else 0
    full = G.sz(0)
    assert L.gcn_aggregate(*before, None, C.byref(full), st) == G.OK and full.value > least
    rows = rng.integers(0, n, 200)
    want, mag = orc.aggregate(og, M, rows=rows, want_mag=True)
    for nbytes in (least, full.value - 1, full.value):
        Z.fill_(float("nan"))
        assert call_sized(G, L.gcn_aggregate, before, st, nbytes) == G.OK, L.gcn_last_error()
        assert_mag_close(host(Z)[rows], want, mag, f"workspace of {nbytes}")
    if least:
        assert call_sized(G, L.gcn_aggregate, before, st, least - 1) == G.E_CAPACITY


def test_layers_with_a_workspace_sized_before_the_graph_was_built(G, orc):
    """A layer's or an epoch's workspace may be sized before the entries of a graph (without a split
    plan) are known; the call takes it."""
    n, fi, fo = 40000, 64, 41
    s, d = gs.chung_lu(n, 4500000, seed=3, dmax=6000.0)
    dg = G.build_csr(n, dev(s), dev(d), split=False)
    rng = np.random.default_rng(1)
    H, W, b = rng.standard_normal((n, fi)), rng.standard_normal((fi, fo)) / 8, rng.standard_normal(fo)
    Hd, Wd, bd = dev(H.astype(np.float32)), dev(W.astype(np.float32)), dev(b.astype(np.float32))
    unbuilt = G.gcn_graph(n, 0, dg.c.nnz_cap, dg.c.row_ptr, dg.c.col_idx, dg.c.deg, dg.c.dinv, dg.c.val)
    Ly = G.make_layer(fi, fo, fi, G.pitch(fo), G.ACT_RELU, 1)
    out, st = G.padded(n, fo), C.c_void_p(torch.cuda.current_stream().cuda_stream)
    L = G.raw_lib()
    fwd = (C.byref(Ly), Hd.data_ptr(), None, Wd.data_ptr(), bd.data_ptr(), out.data_ptr(), None, None, None, None)
    early, full = G.sz(0), G.sz(0)
    assert L.gcn_layer_fwd(C.byref(unbuilt), *fwd, None, C.byref(early), st) == G.OK
    assert L.gcn_layer_fwd(C.byref(dg.c), *fwd, None, C.byref(full), st) == G.OK and full.value > early.value
    assert call_sized(G, L.gcn_layer_fwd, (C.byref(dg.c), *fwd), st, early.value) == G.OK, L.gcn_last_error()
    got = host(out).copy()
    G.layer_fwd(dg, Ly, Hd, None, Wd, bd, out)
    assert_norm_close(got, host(out), "forward, the smaller workspace", 1e-5)
    assert call_sized(G, L.gcn_layer_fwd, (C.byref(dg.c), *fwd), st, early.value - 1) == G.E_CAPACITY
    Gr = dev((rng.standard_normal((n, G.pitch(fo))) / n).astype(np.float32))
    dW, db, Gp = torch.zeros_like(Wd), torch.zeros_like(bd), torch.zeros((n, fi), device="cuda")
    bwd = (C.byref(Ly), Gr.data_ptr(), Hd.data_ptr(), None, None, Wd.data_ptr(), dW.data_ptr(), db.data_ptr(), Gp.data_ptr())
    assert L.gcn_layer_bwd(C.byref(unbuilt), *bwd, None, C.byref(early), st) == G.OK
    assert call_sized(G, L.gcn_layer_bwd, (C.byref(dg.c), *bwd), st, early.value) == G.OK, L.gcn_last_error()
    small = [host(t).copy() for t in (dW, db, Gp)]
    G.layer_bwd(dg, Ly, Gr[:, :fo], Hd, None, None, Wd, dW, db, Gp)
    for a, t in zip(small, (dW, db, Gp)):
        assert_norm_close(a, host(t), "backward, the smaller workspace", 1e-5)
    y = dev(rng.integers(0, fo, n).astype(np.int32))
    losses = []
    for g in (unbuilt, dg.c):
        m = G.Model(n, (fi, fo), [W], [b], ld_x=fi)
        arg = (C.byref(m.c), C.byref(dg.c), Hd.data_ptr(), None, y.data_ptr(), m.loss.data_ptr())
        assert L.gcn_epoch(arg[0], C.byref(g), *arg[2:], None, C.byref(early), st) == G.OK
        assert call_sized(G, L.gcn_epoch, arg, st, early.value) == G.OK, L.gcn_last_error()
        losses.append((float(m.loss), host(m.dW[0])))
    assert losses[0][0] == pytest.approx(losses[1][0], rel=1e-5)
    assert_norm_close(losses[0][1], losses[1][1], "epoch, the smaller workspace", 1e-5)


@pytest.mark.parametrize("csc", [False, True])
def test_feature_views_with_the_counting_workspace(G, orc, csc):
    """The views come out of a workspace without room for the bits of X too (the size that a query
    without the CSR view gives)."""
    n, f = 500, 300
    rng = np.random.default_rng(4)
    X = np.where(rng.random((n, f)) < 0.02, rng.standard_normal((n, f)), 0.0).astype(np.float32)
    Xd, nnz = dev(X), int((X != 0).sum())
    sx, info = G.SparseFeatures(n, f, nnz, "cuda", csc=csc), G.gcn_feature_info()
    L, st = G.raw_lib(), C.c_void_p(torch.cuda.current_stream().cuda_stream)
    head = (Xd.data_ptr(), n, f, f, 4, 5, -1, None, C.byref(info))
    least, full = G.sz(0), G.sz(0)
    assert L.gcn_feature_stats(*head, C.byref(sx.c), None, C.byref(full), st) == G.OK
    if csc:
        least.value = full.value - 4 * n * ((f + 31) // 32)
    else:
        assert L.gcn_feature_stats(*head, None, None, C.byref(least), st) == G.OK
    assert least.value < full.value
    for nbytes in (least.value, full.value):
        sx.c.nnz = nnz
        assert call_sized(G, L.gcn_feature_stats, (*head, C.byref(sx.c)), st, nbytes) == G.OK, L.gcn_last_error()
        rp, col, val = orc.dense_to_csr(X)
        np.testing.assert_array_equal(host(sx.row_ptr), rp)
        np.testing.assert_array_equal(host(sx.col)[:nnz], col)
        np.testing.assert_array_equal(host(sx.val)[:nnz], val.astype(np.float32))
        if csc:
            np.testing.assert_array_equal(host(sx.row)[:nnz], orc.dense_to_csc(X)[1])


@pytest.mark.parametrize("n", [1, 2, 5, 31, 33, 64, 257, 1000, 4093, 4096, 4101, 4124, 4129, 9001])
def test_every_row_is_walked_once(G, orc, n):
    """Workgroups of four rows take their places turned within each eight of them, from 1,024 of them
    on: every row comes out, whatever is left over at the end of the eights."""
    rng = np.random.default_rng(n)
    s, d = messy(rng, n, 5 * n)
    og, dg = orc.build_csr(n, s, d), G.build_csr(n, dev(s), dev(d))
    M = rng.standard_normal((n, 40)).astype(np.float32)
    Z = torch.full((n, 40), float("nan"), device="cuda")
    G.aggregate(dg, dev(M), Z)
    want, mag = orc.aggregate(og, M, want_mag=True)
    assert_mag_close(host(Z), want, mag, f"{n} rows")
    P, arg = orc.aggregate_max(og, M)
    Z.fill_(float("nan"))
    argd = torch.full((n, 40), -7, dtype=torch.int32, device="cuda")
    G.aggregate_max(dg, dev(M), Z, argd)
    np.testing.assert_array_equal(host(Z), P.astype(np.float32))
    np.testing.assert_array_equal(host(argd), arg)
    Z.fill_(float("nan"))
    G.aggregate_max_bwd(dg, dev(M), argd, Z)
    assert_mag_close(host(Z), orc.aggregate_max_backward(og, M, arg), orc.aggregate_max_backward(og, np.abs(M), arg), f"{n} rows, gradient")


def test_blocked_sums_where_rows_miss_blocks(G, orc):
    """Sums blocked by source rows on a graph whose rows have no entry in most blocks, in the first
    one or in the last one (nodes joined to those around them; 100,000 rows, five blocks of 24,576
    or nine of 12,288), with far pairs and a row of all kinds added: every epilogue and the loss."""
    n, k = 100000, 250
    i = np.arange(n, dtype=np.int32)
    s = np.tile(i, k // 2)
    d = np.concatenate([(i + j + 1) % n for j in range(k // 2)]).astype(np.int32)
    rng = np.random.default_rng(2)
    s = np.concatenate([s, np.full(3000, 60000, np.int32), rng.integers(0, n, 5000).astype(np.int32)])
    d = np.concatenate([d, rng.permutation(n)[:3000].astype(np.int32), rng.integers(0, n, 5000).astype(np.int32)])
    og, dg = orc.build_csr(n, s, d), G.build_csr(n, dev(s), dev(d))
    assert og.nnz / n / 9 >= 24
    rows = np.unique(np.concatenate([[0, 1, n - 1, 60000], rng.integers(0, n, 150), np.arange(24500, 24650, 3), s[-5000:-4900]]))
    for w in (33, 128, 200):
        M, b = rng.standard_normal((n, w)).astype(np.float32), rng.standard_normal(w).astype(np.float32)
        mask = rng.standard_normal((n, w)).astype(np.float32)
        ld = (w + 3) // 4 * 4
        Md, Kd = pitched(M, ld), pitched(mask, ld)
        for kind, agg in (("gcn", G.AGG_NORM), ("mean", G.AGG_MEAN), ("mean_t", G.AGG_MEAN_T)):
            want, mag = orc.aggregate(og, M, b, rows=rows, want_mag=True, kind=kind)
            for epi in (G.EPI_NONE, G.EPI_RELU, G.EPI_MASK):
                Z = sentinel(np.zeros((n, w)), ld, 12345.0)
                G.aggregate(dg, Md, Z, bias=dev(b), epi=epi, mask=Kd if epi == G.EPI_MASK else None, agg=agg)
                full = want if epi == G.EPI_NONE else (np.maximum(want, 0) if epi == G.EPI_RELU else want * (mask[rows] > 0))
                assert_mag_close(host(Z)[rows], full, mag, f"{kind} width {w} epi {epi}")
                np.testing.assert_array_equal(padding_of(Z, ld), 12345.0)
        y = rng.integers(0, w, n).astype(np.int32)
        L = G.make_layer(w, w, ld, ld, G.ACT_SOFTMAX_CE, 1)
        out, logits, loss = pitched(np.zeros((n, w)), ld), pitched(np.zeros((n, w)), ld), torch.zeros(1, device="cuda")
        Mf = dev(np.zeros((n, ld), np.float32))
        Mf[:, :w] = dev(M)
        G.layer_fwd(dg, L, Mf[:, :w], None, dev(np.eye(w, dtype=np.float32)), dev(b), out, labels=dev(y), loss=loss, logits=logits)
        want, mag = orc.aggregate(og, M, b, rows=rows, want_mag=True)
        assert_mag_close(host(logits)[rows], want, mag, f"logits {w}")
        assert_norm_close(host(out)[rows] * (n / rows.size), orc.softmax_ce(want, y[rows])[1], f"loss gradient {w}")


@pytest.mark.parametrize("w", [24, 41, 64, 100, 129, 256])
def test_blocked_sums_with_hubs(G, orc, w):
    """Rows so long that their chunks are summed apart from the blocks (beyond 4,096 entries per
    block, two or four here), split rows that are not (5,000 and with four blocks 14,000, and a graph
    without a plan), each epilogue and the loss."""
    n = 40000
    rng = np.random.default_rng(w)
    s, d = gs.chung_lu(n, 4500000, seed=3, dmax=3000.0)
    for hub, ln in ((0, 30000), (7, 14000), (15001, 20000), (n - 1, 5000)):
        s, d = np.concatenate([s, np.full(ln, hub, np.int32)]), np.concatenate([d, rng.permutation(n)[:ln].astype(np.int32)])
    og = orc.build_csr(n, s, d)
    rows = np.unique(np.concatenate([[0, 7, 15001, n - 1], rng.integers(0, n, 150)]))
    M, b = rng.standard_normal((n, w)).astype(np.float32), rng.standard_normal(w).astype(np.float32)
    mask, y = rng.standard_normal((n, w)).astype(np.float32), rng.integers(0, w, n).astype(np.int32)
    ld = (w + 3) // 4 * 4
    Mz = dev(np.zeros((n, ld), np.float32))
    Mz[:, :w] = dev(M)
    for split in (True, False):
        dg = G.build_csr(n, dev(s), dev(d), split=split)
        assert dg.n_long >= 4 or not split
        for kind, agg in (("gcn", G.AGG_NORM), ("mean", G.AGG_MEAN)):
            want, mag = orc.aggregate(og, M, b, rows=rows, want_mag=True, kind=kind)
            for epi in (G.EPI_NONE, G.EPI_RELU, G.EPI_MASK):
                Z = sentinel(np.full((n, w), np.nan), ld, 12345.0)
                G.aggregate(dg, Mz[:, :w], Z, bias=dev(b), epi=epi, mask=pitched(mask, ld) if epi == G.EPI_MASK else None, agg=agg)
                full = want if epi == G.EPI_NONE else (np.maximum(want, 0) if epi == G.EPI_RELU else want * (mask[rows] > 0))
                assert_mag_close(host(Z)[rows], full, mag, f"{kind} width {w} epi {epi} split {split}")
                assert np.isfinite(host(Z)).all()
                np.testing.assert_array_equal(padding_of(Z, ld), 12345.0)
            L = G.make_layer(w, w, ld, ld, G.ACT_SOFTMAX_CE, 1, agg=agg)
            out, logits, loss = pitched(np.zeros((n, w)), ld), pitched(np.zeros((n, w)), ld), torch.zeros(1, device="cuda")
            G.layer_fwd(dg, L, Mz[:, :w], None, dev(np.eye(w, dtype=np.float32)), dev(b), out, labels=dev(y), loss=loss, logits=logits)
            assert_mag_close(host(logits)[rows], want, mag, f"logits {kind} {w} split {split}")
            assert_norm_close(host(out)[rows] * (n / rows.size), orc.softmax_ce(want, y[rows])[1], f"loss gradient {kind} {w} split {split}")


@pytest.mark.parametrize("n,e", [(33000, 40000), (33000, 600000), (70000, 150000), (140000, 11500000)])
def test_narrow_rows_by_groups_and_wavefronts(G, orc, n, e):
    """Up to 16 columns the rows go to lane groups, which share long rows (up to 8 columns), or to one
    wavefront each, by the rows per graph and the entries per row: both sides of the lines, rows of
    a few hundred to a few thousand entries among short ones, split rows, every epilogue, the loss,
    bit for bit the same with and without the row order."""
    s, d = gs.chung_lu(n, e, seed=7, dmax=n / 8.0)
    rng = np.random.default_rng(e)
    for hub, ln in ((1, 900), (2, 3000), (n - 1, 4090), (n // 2, 6000)):
        s, d = np.concatenate([s, np.full(ln, hub, np.int32)]), np.concatenate([d, rng.permutation(n)[:ln].astype(np.int32)])
    og, dg = orc.build_csr(n, s, d), G.build_csr(n, dev(s), dev(d))
    plain = G.build_csr(n, dev(s), dev(d), order=False)
    rows = np.unique(np.concatenate([[0, 1, 2, n // 2, n - 1], rng.integers(0, n, 200), np.argsort(og.deg)[-30:]]))
    for w in (1, 4, 5, 8, 9, 16):
        M, b = rng.standard_normal((n, w)).astype(np.float32), rng.standard_normal(w).astype(np.float32)
        mask, y = rng.standard_normal((n, w)).astype(np.float32), rng.integers(0, w, n).astype(np.int32)
        ld = (w + 3) // 4 * 4
        Md, Kd = sentinel(M, ld, 7.0), pitched(mask, ld)
        for kind, agg, epi in (("gcn", G.AGG_NORM, G.EPI_NONE), ("mean", G.AGG_MEAN, G.EPI_RELU), ("mean_t", G.AGG_MEAN_T, G.EPI_MASK)):
            outs = []
            for g in (dg, plain):
                Z = sentinel(np.full((n, w), np.nan), ld, 12345.0)
                G.aggregate(g, Md, Z, bias=dev(b), epi=epi, mask=Kd if epi == G.EPI_MASK else None, agg=agg)
                np.testing.assert_array_equal(padding_of(Z, ld), 12345.0)
                outs.append(host(Z))
            np.testing.assert_array_equal(*outs)
            want, mag = orc.aggregate(og, M, b, rows=rows, want_mag=True, kind=kind)
            want = want if epi == G.EPI_NONE else (np.maximum(want, 0) if epi == G.EPI_RELU else want * (mask[rows] > 0))
            assert_mag_close(outs[0][rows], want, mag, f"{kind} {n} rows width {w} epi {epi}")
        L = G.make_layer(w, w, ld, ld, G.ACT_SOFTMAX_CE, 1)
        out, logits, loss = pitched(np.zeros((n, w)), ld), pitched(np.zeros((n, w)), ld), torch.zeros(1, device="cuda")
        G.layer_fwd(dg, L, Md, None, dev(np.eye(w, dtype=np.float32)), dev(b), out, labels=dev(y), loss=loss, logits=logits)
        want, mag = orc.aggregate(og, M, b, rows=rows, want_mag=True)
        assert_mag_close(host(logits)[rows], want, mag, f"logits {n} rows width {w}")
        assert_norm_close(host(out)[rows] * (n / rows.size), orc.softmax_ce(want, y[rows])[1], f"loss gradient {n} rows width {w}")


def test_spmm_row_beyond_31_bits(G):
    """gcn_spmm over a row of 2^31 + 9 entries (columns may repeat) among short ones."""
    long_row, n = (1 << 31) + 9, 8
    ln = torch.ones(n, dtype=torch.int64, device="cuda")
    ln[3] = long_row
    ptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    ptr[1:] = ln.cumsum(0)
    note("a row of 2^31 + 9 entries")
    nnz = int(ptr[-1])
    idx, val = torch.zeros(nnz, dtype=torch.int32, device="cuda"), torch.ones(nnz, device="cuda")
    val[-1] = 5.0
    B = torch.tensor([[1.0, 2.0, 0.0, -1.0], [9.0, 9.0, 9.0, 9.0]], device="cuda")
    out = torch.full((n, 4), float("nan"), device="cuda")
    G.spmm(ptr, idx, val, B, out)
    want = np.tile([1.0, 2.0, 0.0, -1.0], (n, 1))
    want[3] *= long_row
    want[n - 1] *= 5.0
    np.testing.assert_allclose(host(out), want, rtol=1e-5)


@pytest.mark.parametrize("f,ld", [(1, 4), (5, 8), (32, 32), (33, 36), (61, 64), (64, 68), (65, 68), (127, 128), (128, 128)])
def test_feature_views_narrow_rows(G, orc, f, ld):
    """Rows of up to 128 columns, several to a wavefront: counts, bits and views byte for byte, few
    rows and more than one turn of the grid, empty and full rows, NaN in the padding; dense rows of
    the column view read four turns at a time (more than 64 nonzeros)."""
    rng = np.random.default_rng(f)
    for n, p in ((1, 1.0), (7, 0.5), (70001 if f > 8 else 600001, 0.03), (3000, 0.9)):
        X = np.where(rng.random((n, f)) < p, rng.standard_normal((n, f)), 0.0).astype(np.float32)
        X[n // 2] = np.inf
        X[n - 1, f - 1] = -0.0
        rnd = torch.zeros(n, dtype=torch.int64, device="cuda")
        info, sx = G.feature_stats(pitched(X, ld), materialize=True, row_nnz=rnd)
        nnz = int((X != 0).sum())
        assert info["nnz"] == nnz
        np.testing.assert_array_equal(host(rnd), (X != 0).sum(1))
        for got, want in zip((sx.row_ptr, sx.col, sx.val), orc.dense_to_csr(X)):
            np.testing.assert_array_equal(host(got)[:want.size], want)
        for got, want in zip((sx.col_ptr, sx.row, sx.cval), orc.dense_to_csc(X)):
            np.testing.assert_array_equal(host(got)[:want.size], want)


@pytest.mark.parametrize("w", [40, 128])
def test_tune_row_order_keeps_what_it_cannot_time(G, w):
    """An aggregation that takes the rows as they come cannot tell whether the order pays: the tuner
    keeps it, every time."""
    wl = gs.WORKLOADS["cora_like"]
    s, d = gs.make_graph(wl)
    for _ in range(20):
        g = G.build_csr(wl.n, dev(s), dev(d))
        assert G.tune_row_order(g, w) and g.order is not None and g.c.order == g.order.data_ptr()


@pytest.mark.parametrize("n,e,widths", [(140000, 5900000, (17, 24, 32)), (140000, 1400000, (130, 200, 246)), (40000, 800000, (65, 96, 128, 256))])
def test_plans_of_larger_graphs(G, orc, n, e, widths):
    """The forms that only larger graphs take, checked on sampled rows: sums of rows of one line
    blocked by source rows (from 131,072 rows on; every slice of a wavefront keeps a row of its own
    for the loss), two panels of rows that share lines by lane groups in the row order, panels of 32
    columns."""
    s, d = gs.chung_lu(n, e, seed=9, dmax=6000.0)
    og, dg = orc.build_csr(n, s, d), G.build_csr(n, dev(s), dev(d))
    plain = G.build_csr(n, dev(s), dev(d), order=False)
    avg = og.nnz / n
    assert {17: avg >= 72, 130: 12 <= avg < 24, 65: avg >= 32}[widths[0]], avg
    rng = np.random.default_rng(n + e)
    rows = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 150), np.argsort(og.deg)[-20:], np.argsort(og.deg)[:20]]))
    for w in widths:
        ld = G.pitch(w)
        M, b = rng.standard_normal((n, w)).astype(np.float32), rng.standard_normal(w).astype(np.float32)
        mask, y = rng.standard_normal((n, w)).astype(np.float32), rng.integers(0, w, n).astype(np.int32)
        Md, Kd = sentinel(M, ld, 7.0), pitched(mask, ld)
        for kind, agg, epi in (("gcn", G.AGG_NORM, G.EPI_NONE), ("mean", G.AGG_MEAN, G.EPI_RELU), ("sum", G.AGG_SUM, G.EPI_MASK)):
            outs = []
            for g in (dg, plain):
                Z = sentinel(np.full((n, w), np.nan), ld, 12345.0)
                G.aggregate(g, Md, Z, bias=dev(b), epi=epi, mask=Kd if epi == G.EPI_MASK else None, agg=agg)
                np.testing.assert_array_equal(padding_of(Z, ld), 12345.0)
                outs.append(host(Z))
            np.testing.assert_array_equal(*outs)
            want, mag = orc.aggregate(og, M, b, rows=rows, want_mag=True, kind=kind)
            want = want if epi == G.EPI_NONE else (np.maximum(want, 0) if epi == G.EPI_RELU else want * (mask[rows] > 0))
            assert_mag_close(outs[0][rows], want, mag, f"{kind} {n} rows width {w} epi {epi}")
        L = G.make_layer(w, w, ld, ld, G.ACT_SOFTMAX_CE, 1)
        out, logits, loss = sentinel(np.zeros((n, w)), ld, 12345.0), sentinel(np.zeros((n, w)), ld, 12345.0), torch.zeros(1, device="cuda")
        G.layer_fwd(dg, L, Md, None, dev(np.eye(w, dtype=np.float32)), dev(b), out, labels=dev(y), loss=loss, logits=logits)
        want, mag = orc.aggregate(og, M, b, rows=rows, want_mag=True)
        assert_mag_close(host(logits)[rows], want, mag, f"logits {n} rows width {w}")
        assert_norm_close(host(out)[rows] * (n / rows.size), orc.softmax_ce(want, y[rows])[1], f"loss gradient {n} rows width {w}")
        np.testing.assert_array_equal(padding_of(out, ld), 12345.0)
