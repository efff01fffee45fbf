"""GPU parity of the combination step Y = act(A * W) (aires_spmm, Sec. II-A
Eq. 3) through the C-ABI against the oracle's double-precision product.

Bar: every entry within the fp32 summation error bound of the GPU's
arbitrary order with fused multiply-adds,
    |y - y64| <= (n_i + 2) * 2^-24 * sum_k |a_ik w_kj| + 2^-24 * |y64|,
where n_i is the number of stored entries of row i (the standard bound
gamma_n for a sum of n_i rounded terms, plus the final rounding); exact
(bit-equal to the integer product) when every value is a small integer.
Both kernel families are held to it: the entry gather ("rows") and the
densified tiles on the matrix cores ("dense_tiles"), whose extra products
with absent entries are exact zeros for finite W."""
import numpy as np
import pytest

import oracle
import workloads
from workloads import CSR

pytestmark = pytest.mark.gpu

U = 2.0 ** -24
ALGOS = ["rows", "dense_tiles"]


@pytest.fixture(scope="module")
def torch_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch


def say(msg):
    print("[gpu-case] " + msg, flush=True)


def dev_csr(torch, A, rp64=False, a_offset=0):
    """A on the device; a_offset > 0 starts its column and value arrays that
    many elements into their allocations (off 16-byte alignment for 1-3)."""
    rp = A.rp.astype(np.int64 if rp64 else np.int32)
    col = torch.zeros(A.nnz + a_offset, dtype=torch.int32, device="cuda")[a_offset:]
    val = torch.zeros(A.nnz + a_offset, dtype=torch.float32, device="cuda")[a_offset:]
    col.copy_(torch.from_numpy(A.col.astype(np.int32)))
    val.copy_(torch.from_numpy(A.val.astype(np.float32)))
    return (A.nrows, A.ncols, torch.from_numpy(rp).cuda(), col, val)


def check(torch, A, W, relu=False, rp64=False, ldw_pad=0, ldy_pad=0, w_offset=0, exact=False, name="",
          algo="auto", a_offset=0):
    import paper_2507_02006_amd as aires
    say("%s algo=%s m=%d K=%d F=%d relu=%d rp64=%d pads=(%d,%d) off=%d a_off=%d" % (
        name, algo, A.nrows, A.ncols, W.shape[1], relu, rp64, ldw_pad, ldy_pad, w_offset, a_offset))
    K, F = W.shape
    buf = torch.zeros(K * (F + ldw_pad) + w_offset + 1, dtype=torch.float32, device="cuda")
    Wd = buf[w_offset:w_offset + K * (F + ldw_pad)].view(K, F + ldw_pad)[:, :F]
    Wd.copy_(torch.from_numpy(W))
    ybuf = torch.full((A.nrows, F + ldy_pad), 7.0, dtype=torch.float32, device="cuda")
    Y = aires.spmm(dev_csr(torch, A, rp64, a_offset), Wd, relu=relu, out=ybuf[:, :F], algo=algo)
    torch.cuda.synchronize()
    y = Y.cpu().numpy().astype(np.float64)
    if ldy_pad:
        assert np.all(ybuf[:, F:].cpu().numpy() == 7.0), "columns past F were written"
    ref, refabs = oracle.spmm(A, W, relu=relu)
    if exact:
        assert np.array_equal(y, ref), name
        return
    n = np.diff(A.rp.astype(np.int64))[:, None]
    tol = (n + 2) * U * refabs + U * np.abs(ref)
    err = np.abs(y - ref)
    bad = err > tol
    assert not bad.any(), "%s: %d entries over the bound, worst %g" % (name, bad.sum(), (err - tol).max())


@pytest.mark.parametrize("algo", ALGOS)
@pytest.mark.parametrize("F", [1, 7, 64, 65, 100, 128, 129, 200, 256, 512, 700])
def test_widths(torch_gpu, F, algo):
    """Rows: lane groups of 16-byte loads up to 64 lanes wide, one column a
    lane below four columns; 512 and 700 take several column blocks; where F
    is not a multiple of four the last lane's vector is moved back.
    Dense tiles: 64- or 128-column tiles, ragged in m (300), K (90) and F."""
    rng = np.random.default_rng(F)
    A = workloads.random_csr(rng, 300, 90, 0.05)
    W = rng.uniform(-1, 1, (90, F)).astype(np.float32)
    check(torch_gpu, A, W, name="width %d" % F, algo=algo)


@pytest.mark.parametrize("algo", ALGOS)
@pytest.mark.parametrize("relu", [False, True])
def test_integer_values_exact(torch_gpu, relu, algo):
    """Small integers: every product and partial sum is exact in fp32, so Y
    equals the integer product whatever the order."""
    rng = np.random.default_rng(5)
    Ad = rng.integers(-3, 4, (257, 129)) * (rng.random((257, 129)) < 0.1)
    A = CSR(257, 129, *_csr_parts(Ad))
    W = rng.integers(-3, 4, (129, 96)).astype(np.float32)
    check(torch_gpu, A, W, relu=relu, exact=True, name="integer relu=%d" % relu, algo=algo)


def _csr_parts(D):
    rows, cols = np.nonzero(D)
    rp = np.zeros(D.shape[0] + 1, dtype=np.int64)
    np.add.at(rp, rows + 1, 1)
    return np.cumsum(rp).astype(np.int32), cols.astype(np.int32), D[rows, cols].astype(np.float32)


@pytest.mark.parametrize("algo", ALGOS)
def test_heavy_rows_split_over_a_workgroup(torch_gpu, algo):
    """Rows above the limit for one wavefront take the eight wavefronts of a
    workgroup (and an LDS reduction); mixed with light and empty rows.  For dense
    tiles, rows with more than 32 entries in a 64-column chunk take several
    load rounds."""
    rng = np.random.default_rng(7)
    K = 3000
    lens = np.array([0, 3, 513, 512, 2999, 0, 1, 1500, 700, 5] * 4)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col = np.concatenate([np.sort(rng.choice(K, L, replace=False)) for L in lens]).astype(np.int32)
    val = rng.uniform(-1, 1, len(col)).astype(np.float32)
    A = CSR(len(lens), K, rp, col, val)
    for F in (64, 256, 600):
        W = rng.uniform(-1, 1, (K, F)).astype(np.float32)
        check(torch_gpu, A, W, relu=True, name="heavy F=%d" % F, algo=algo)


@pytest.mark.parametrize("F", [2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 128, 129, 192, 256, 257, 384, 512, 516, 2100])
def test_rows_lane_groups_and_column_blocks(torch_gpu, F):
    """Entry gather: every lane-group width (F around powers of two), vectors
    moved back at the end of a row, one, two and more column blocks (more
    than the XCDs at 2100), and row lengths around a batch of 64, the
    workgroup limit (256) and the eight wavefronts' turn (512), with strides
    that keep whole cache lines and one that does not."""
    rng = np.random.default_rng(1000 + F)
    K = 1400
    lens = np.array([0, 1, 2, 7, 8, 9, 31, 33, 63, 64, 65, 129, 255, 256, 257, 300, 512, 513, 1025, 1400, 0])
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    col = np.concatenate([np.sort(rng.choice(K, L, replace=False)) for L in lens]).astype(np.int32)
    A = CSR(len(lens), K, rp, col, rng.uniform(-1, 1, len(col)).astype(np.float32))
    W = rng.uniform(-1, 1, (K, F)).astype(np.float32)
    check(torch_gpu, A, W, name="lane groups F=%d" % F, algo="rows")
    check(torch_gpu, A, W, relu=True, rp64=True, ldw_pad=(1 if F % 32 == 0 else 32 - F % 32), ldy_pad=3,
          name="lane groups padded F=%d" % F, algo="rows")
    Wn = W.copy()  # a row of W that no entry names may hold anything
    sub = CSR(12, K, rp[:13], col[:rp[12]], A.val[:rp[12]])
    Wn[np.setdiff1d(np.arange(K), sub.col)] = np.nan
    import paper_2507_02006_amd as aires
    y = aires.spmm(dev_csr(torch_gpu, sub), torch_gpu.from_numpy(Wn).cuda(), algo="rows")
    assert torch_gpu.isfinite(y).all()


def rows_of(rng, lens, K):
    """A CSR of these row lengths, one entry in each of as many equal parts
    of the K columns, small integer values."""
    lens = np.asarray(lens)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    at = np.arange(rp[-1]) - np.repeat(rp[:-1], lens)
    L = np.repeat(lens, lens)
    lo, hi = at * K // L, (at + 1) * K // L
    col = (lo + rng.integers(0, 1 << 30, len(at)) % (hi - lo)).astype(np.int32)
    return CSR(len(lens), K, rp.astype(np.int32), col, rng.integers(-3, 4, len(at)).astype(np.float32))


@pytest.mark.parametrize("F", [3, 64, 256, 516])
def test_many_long_rows(torch_gpu, F):
    """Long rows in every count: few (a group of rows each), many of like
    length (the limit rises with the mean: a wavefront each), those with hubs
    among them that stay split, and a ragged last group; integer values, so
    the result is exact."""
    rng = np.random.default_rng(40 + F)
    K = 2048
    mixed = rng.integers(250, 420, 3000)
    mixed[rng.choice(3000, 40, replace=False)] = K
    for lens in ([300] * 9, [K] * 65, [900] * 257, [257] * 700 + [3] * 400, mixed):
        A = rows_of(rng, lens, K)
        check(torch_gpu, A, rng.integers(-3, 4, (K, F)).astype(np.float32), relu=F == 64, rp64=F == 256, exact=True,
              name="%d long rows F=%d" % (len(lens), F), algo="rows")


@pytest.mark.parametrize("F", [64, 256])
@pytest.mark.parametrize("m", [256, 4000, 20000])
def test_many_long_rows_cost(torch_gpu, m, F):
    """An entry costs about as much in rows just above the limit where rows
    are split as in rows below it, however many there are (at most four times:
    they were 15 to 40 times as dear while a workgroup looked through 512 rows
    whatever their number)."""
    import paper_2507_02006_amd as aires
    rng = np.random.default_rng(m + F)
    K = 4096
    W = torch_gpu.from_numpy(rng.uniform(-1, 1, (K, F)).astype(np.float32)).cuda()
    Y = torch_gpu.empty((m, F), device="cuda")
    cost = {}
    for L in (250, 300, 900):
        A = dev_csr(torch_gpu, rows_of(rng, [L] * m, K))
        best = float("inf")
        for _ in range(5):
            a, b = (torch_gpu.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                aires.spmm(A, W, out=Y, algo="rows")
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        cost[L] = best / L
    say("long rows m=%d F=%d: ns per call and entry of a row %s" % (m, F, {L: round(c * 2e5) for L, c in cost.items()}))
    assert max(cost.values()) <= 4 * cost[250]


@pytest.mark.parametrize("F", [(1 << 21) + 69, (1 << 26) + 5, (1 << 31) - 1])
def test_widest_rows(torch_gpu, F):
    """More columns than a launch takes, with split and light rows; so many
    that one launch with workgroups for all their blocks was refused; and the
    widest F there is: integer values, so the result is exact."""
    import paper_2507_02006_amd as aires
    torch = torch_gpu
    lens = {21: [260, 3, 0, 259], 26: [2, 0, 1]}.get(F.bit_length() - 1, [1, 0])
    K = max(lens)
    rng = np.random.default_rng(F % 1000)
    A = rows_of(rng, lens, K)
    say("widest F=%d" % F)
    W = torch.empty((K, F), device="cuda")
    for k in range(K):
        W[k] = (torch.arange(F, device="cuda", dtype=torch.int32) * (2 * k + 1) >> 3) % 7 - 3
    Y = aires.spmm(dev_csr(torch, A), W, algo="rows")
    for i in range(A.nrows):
        y = torch.zeros(F, device="cuda")
        for e in range(A.rp[i], A.rp[i + 1]):
            y.add_(W[int(A.col[e])], alpha=float(A.val[e]))
        assert torch.equal(Y[i], y), i
        del y
    del W, Y
    torch.cuda.empty_cache()


@pytest.mark.parametrize("algo", ALGOS)
def test_strides_offsets_and_rp64(torch_gpu, algo):
    """Row strides above F (padding untouched), a W base that is not
    vector-aligned, and 64-bit row pointers."""
    rng = np.random.default_rng(8)
    A = workloads.random_csr(rng, 200, 70, 0.1)
    W = rng.uniform(-1, 1, (70, 256)).astype(np.float32)
    check(torch_gpu, A, W, ldw_pad=3, ldy_pad=5, name="pads", algo=algo)
    check(torch_gpu, A, W, ldw_pad=4, name="aligned pad", algo=algo)
    check(torch_gpu, A, W, w_offset=1, name="unaligned W", algo=algo)
    check(torch_gpu, A, W, rp64=True, relu=True, name="rp64", algo=algo)
    for off in (1, 2, 4):  # A's arrays off 16-byte alignment (single-entry loads), then back on it
        check(torch_gpu, A, W, a_offset=off, name="A offset %d" % off, algo=algo)


def test_edges(torch_gpu):
    import paper_2507_02006_amd as aires
    torch = torch_gpu
    rng = np.random.default_rng(9)
    E = CSR(6, 10, np.zeros(7, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32))
    W = rng.uniform(-1, 1, (10, 33)).astype(np.float32)
    for algo in ALGOS:
        check(torch, E, W, name="all rows empty", algo=algo)
    check(torch, CSR(5, 0, np.zeros(6, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32)),
          np.zeros((0, 20), np.float32), name="K = 0", algo="dense_tiles")
    Y = aires.spmm(dev_csr(torch, CSR(0, 10, np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32))),
                   torch.from_numpy(W).cuda())
    assert Y.shape == (0, 33)
    A = workloads.random_csr(rng, 8, 10, 0.5)
    Y = aires.spmm(dev_csr(torch, A), torch.zeros((10, 0), device="cuda"))
    assert Y.shape == (8, 0)
    with pytest.raises(ValueError):
        aires.spmm(dev_csr(torch, A), torch.zeros((11, 4), device="cuda"))
    with pytest.raises(ValueError):
        aires.spmm(dev_csr(torch, A), torch.zeros((10, 4), device="cuda"), algo="gemm")


@pytest.mark.parametrize("density", [0.3, 1.0])
def test_dense_tiles_dense_rows(torch_gpu, density):
    """Fully dense and 30 % rows: 64 entries per 64-column chunk (two load
    rounds of 32 and a third that finds the chunk's end), K not a multiple
    of 64, several column tiles on the XCD-ordered grid."""
    rng = np.random.default_rng(int(density * 10))
    A = workloads.random_csr(rng, 517, 333, density)
    for F in (48, 300):
        W = rng.uniform(-1, 1, (333, F)).astype(np.float32)
        check(torch_gpu, A, W, relu=True, name="dense rows %.1f F=%d" % (density, F), algo="dense_tiles")
        check(torch_gpu, A, W, name="dense rows %.1f F=%d A offset 1" % (density, F), algo="dense_tiles",
              a_offset=1)


@pytest.mark.parametrize("K", [1, 8, 9, 31, 32, 33, 63, 64, 65, 97])
def test_dense_tiles_chunk_edges(torch_gpu, K):
    """One, two and more 32-wide chunks with every kind of remainder, for
    tiles staged after (F <= 64) and between (above) the products of a
    chunk; the bar is check()'s summation bound."""
    rng = np.random.default_rng(500 + K)
    A = workloads.random_csr(rng, 131, K, 0.5)
    for F in (64, 65, 132):
        W = rng.uniform(-1, 1, (K, F)).astype(np.float32)
        check(torch_gpu, A, W, relu=F == 132, rp64=F == 65, name="chunk edges K=%d F=%d" % (K, F), algo="dense_tiles")


def test_dense_tiles_grid_loop(torch_gpu):
    """More tiles than the grid (65536 blocks): the second sweep of the
    persistent loop, checked on sampled rows and the last rows (1 075 200
    rows, one entry each, K = 16, F = 512: 67200 tiles)."""
    import paper_2507_02006_amd as aires
    torch = torch_gpu
    rng = np.random.default_rng(12)
    m, K, F = 1075200, 16, 512
    rp = np.arange(m + 1, dtype=np.int32)
    col = (np.arange(m) * 7 % K).astype(np.int32)
    val = rng.integers(-4, 5, m).astype(np.float32)
    A = CSR(m, K, rp, col, val)
    W = rng.integers(-8, 9, (K, F)).astype(np.float32)
    say("grid loop m=%d K=%d F=%d" % (m, K, F))
    Y = aires.spmm(dev_csr(torch, A), torch.from_numpy(W).cuda(), algo="dense_tiles")
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([rng.integers(0, m, 2000), np.arange(m - 3000, m)]))
    y = Y[torch.from_numpy(rows).cuda()].cpu().numpy().astype(np.float64)
    sub = CSR(len(rows), K, np.arange(len(rows) + 1, dtype=np.int32), col[rows], val[rows])
    ref, _ = oracle.spmm(sub, W)
    assert np.array_equal(y, ref)


def test_gcn_layer_on_aggregated_features(torch_gpu):
    """A GCN layer H' = relu((A_norm X) W) (Eqs. 1-3): the aggregation from
    aires_spgemm, then the combination on its CSR output (int64 row
    pointers), against the oracle on the oracle's aggregation."""
    import paper_2507_02006_amd as aires
    torch = torch_gpu
    A, X = workloads.workload(2, n=8192)  # cfg2 scaled down: F_in = 512 features at 5 %
    rng = np.random.default_rng(10)
    W = rng.uniform(-0.5, 0.5, (X.ncols, 64)).astype(np.float32)
    say("gcn layer m=%d nnzA=%d F_in=%d F_out=64" % (A.nrows, A.nnz, X.ncols))
    with aires.tile_plan(aires.to_device(A), aires.to_device(X), 0) as plan:
        C = aires.spgemm(plan)
        Wd = torch.from_numpy(W).cuda()
        H = aires.spmm((C.nrows, C.ncols, C.rp, C.col, C.val), Wd, relu=True)
        torch.cuda.synchronize()
        h = H.cpu().numpy().astype(np.float64)
    Co = oracle.spgemm(A, X)
    ref, refabs = oracle.spmm(CSR(Co.r1 - Co.r0, Co.ncols, Co.rp, Co.col, Co.val), W, relu=True)
    # C itself differs from the oracle's by at most 1e-5 (1 + |c|) per entry
    n = np.diff(Co.rp)[:, None]
    cabs, _ = oracle.spmm(CSR(Co.r1 - Co.r0, Co.ncols, Co.rp, Co.col, np.abs(Co.val)), np.abs(W))
    tol = (n + 2) * U * refabs + U * np.abs(ref) + 1e-5 * (np.abs(W).sum(0)[None, :] + cabs)
    assert np.all(np.abs(h - ref) <= tol)


@pytest.mark.slow
@pytest.mark.parametrize("algo", ALGOS)
def test_full_cfg2_combination_sampled(torch_gpu, algo):
    """The combination step at the size the bench times: relu(C W) with C
    the aggregate of the full cfg2 (262144 x 512, 39.2 M entries) from
    aires_spgemm and W 512 x 256, checked on sampled rows and the heaviest
    rows against the oracle's product of the oracle's aggregate rows."""
    import paper_2507_02006_amd as aires
    torch = torch_gpu
    A, X = workloads.workload(2)
    rng = np.random.default_rng(21)
    W = rng.uniform(-0.05, 0.05, (X.ncols, 256)).astype(np.float32)
    say("full cfg2 combination algo=%s" % algo)
    with aires.tile_plan(aires.to_device(A), aires.to_device(X), 0) as plan:
        C = aires.spgemm(plan)
        H = aires.spmm((C.nrows, C.ncols, C.rp, C.col, C.val), torch.from_numpy(W).cuda(), relu=True, algo=algo)
        torch.cuda.synchronize()
        crow = np.diff(C.rp.cpu().numpy())
        rows = np.unique(np.concatenate([rng.choice(A.nrows, 200, replace=False), np.argsort(crow)[-5:],
                                         [0, A.nrows - 1]]))
        h = H[torch.from_numpy(rows).cuda()].cpu().numpy().astype(np.float64)
    for r, hr in zip(rows, h):
        Co = oracle.spgemm(A, X, int(r), int(r) + 1)
        row = CSR(1, Co.ncols, Co.rp, Co.col, Co.val)
        ref, refabs = oracle.spmm(row, W, relu=True)
        cabs, _ = oracle.spmm(CSR(1, Co.ncols, Co.rp, Co.col, np.abs(Co.val)), np.abs(W))
        n = len(Co.col)
        tol = (n + 2) * U * refabs + U * np.abs(ref) + 1e-5 * (np.abs(W).sum(0)[None, :] + cabs)
        assert np.all(np.abs(hr[None, :] - ref) <= tol), "row %d" % r
