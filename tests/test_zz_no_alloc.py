"""The allocation-free entry point (aires_spgemm_noalloc) against the
allocating one (aires_spgemm) on the same plans, through the C-ABI: two
calls in a row, the second on a smaller input (the fixed workspace keeps
the first call's contents), narrow and wide products; C arrays too small
and a workspace beyond the fixed array give AIRES_E_CAPACITY."""
import numpy as np
import pytest

import workloads
from workloads import CSR

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.fixture(scope="module")
def torch_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch


def say(msg):
    print("[gpu-case] " + msg, flush=True)


def _pair(torch, A, B, **kw):
    """(allocating result, allocation-free result) on one plan."""
    import paper_2507_02006_amd as aires
    dA, dB = aires.to_device(A), aires.to_device(B)
    with aires.tile_plan(dA, dB, 0, **kw) as plan:
        C = aires.spgemm(plan)
        torch.cuda.synchronize()
        want = (C.rp.cpu().numpy(), C.col.cpu().numpy(), C.val.cpu().numpy())
        del C
        rp = torch.full((A.nrows + 1,), -1, dtype=torch.int64, device="cuda")
        cap = len(want[1]) + 17
        col = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
        val = torch.full((cap,), float("nan"), dtype=torch.float32, device="cuda")
        nnz = aires.spgemm_noalloc(plan, rp, col, val)
        torch.cuda.synchronize()
        got = (rp.cpu().numpy(), col[:nnz].cpu().numpy(), val[:nnz].cpu().numpy())
        # nothing is written past nnz(C)
        assert np.all(col[nnz:].cpu().numpy() == -1)
    return want, got


def _same(want, got):
    assert np.array_equal(want[0], got[0]), "row_ptr differs"
    assert np.array_equal(want[1], got[1]), "col_idx differs"
    w = want[2].astype(np.float64)
    assert np.all(np.abs(got[2] - w) <= TOL * (1 + np.abs(w))), "values differ"


@pytest.mark.parametrize("case", ["narrow", "wide"])
def test_noalloc_matches_spgemm_twice(torch_gpu, case):
    if case == "narrow":
        big = workloads.workload(2, n=32768)
        small = workloads.workload(1, n=2048)
        kw = dict(split_min_products=4096, max_tile_rows=10000)
    else:
        big = workloads.workload(3, n=24000)
        small = workloads.workload(3, n=5000)
        kw = dict(dense_max_cols=2048, window_grain_cols=2048, max_tile_rows=7000)
    for name, (A, B) in (("first", big), ("second, smaller", small)):
        say("noalloc %s %s: m=%d N=%d nnzA=%d" % (case, name, A.nrows, B.ncols, A.nnz))
        want, got = _pair(torch_gpu, A, B, **kw)
        _same(want, got)


def test_noalloc_capacity(torch_gpu):
    """C arrays too small: AIRES_E_CAPACITY with nnz(C) and C.row_ptr
    valid; a repeat with arrays of that size succeeds."""
    import paper_2507_02006_amd as aires
    from paper_2507_02006_amd import _binding as B_
    torch = torch_gpu
    A, B = workloads.workload(1, n=3000)
    dA, dB = aires.to_device(A), aires.to_device(B)
    with aires.tile_plan(dA, dB, 0) as plan:
        C = aires.spgemm(plan)
        torch.cuda.synchronize()
        want = (C.rp.cpu().numpy(), C.col.cpu().numpy(), C.val.cpu().numpy())
        rp = torch.empty(A.nrows + 1, dtype=torch.int64, device="cuda")
        col = torch.empty(10, dtype=torch.int32, device="cuda")
        val = torch.empty(10, dtype=torch.float32, device="cuda")
        with pytest.raises(aires.AiresError) as e:
            aires.spgemm_noalloc(plan, rp, col, val)
        torch.cuda.synchronize()
        assert e.value.status == B_.E_CAPACITY and e.value.nnz == len(want[1])
        assert np.array_equal(rp.cpu().numpy(), want[0])
        n = e.value.nnz
        col = torch.empty(n, dtype=torch.int32, device="cuda")
        val = torch.empty(n, dtype=torch.float32, device="cuda")
        assert aires.spgemm_noalloc(plan, rp, col, val) == n
        torch.cuda.synchronize()
        _same(want, (rp.cpu().numpy(), col.cpu().numpy(), val.cpu().numpy()))


def test_noalloc_workspace_too_large(torch_gpu):
    """8 M rows need 96 MB of row workspace: more than the fixed 64 MiB
    array, so the call is refused before any kernel runs."""
    import paper_2507_02006_amd as aires
    from paper_2507_02006_amd import _binding as B_
    torch = torch_gpu
    m = 8 << 20
    A = CSR(m, 8, np.arange(m + 1, dtype=np.int32), np.zeros(m, np.int32), np.ones(m, np.float32))
    B = CSR(8, 8, np.arange(9, dtype=np.int32), np.arange(8, dtype=np.int32), np.ones(8, np.float32))
    with aires.tile_plan(aires.to_device(A), aires.to_device(B), 0) as plan:
        rp = torch.empty(m + 1, dtype=torch.int64, device="cuda")
        col = torch.empty(m, dtype=torch.int32, device="cuda")
        val = torch.empty(m, dtype=torch.float32, device="cuda")
        with pytest.raises(aires.AiresError) as e:
            aires.spgemm_noalloc(plan, rp, col, val)
        assert e.value.status == B_.E_CAPACITY and "scratch" in str(e.value)
        assert e.value.nnz == -1


def _rows_of(rng, lens, ncols):
    """Rows of these lengths, one entry in each of as many equal parts of the
    columns, small integer values."""
    lens = np.asarray(lens)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    at = np.arange(rp[-1]) - np.repeat(rp[:-1], lens)
    L = np.repeat(lens, lens)
    lo, hi = at * ncols // L, (at + 1) * ncols // L
    col = (lo + rng.integers(0, 1 << 30, len(at)) % (hi - lo)).astype(np.int32)
    return CSR(len(lens), ncols, rp, col, rng.integers(-3, 4, len(at)).astype(np.float32))


@pytest.mark.parametrize("m,N,mean", [(16000, 64, 6), (100000, 200, 20), (60000, 512, 20), (30000, 2000, 12)])
def test_noalloc_keeps_the_bitmap_path(torch_gpu, m, N, mean):
    """C lies in the caller's arrays, so its size says nothing about the fixed
    workspace: an allocation-free call whose C is larger than what is left of
    that keeps the bitmaps it has made.  Rows of few products and rows of 2000
    take a bin each there, and are one bin of the general path, which runs all
    of its bins where it takes over late: the launches of the numeric phase say
    which one ran.  Integer values, so both calls are exact."""
    import paper_2507_02006_amd as aires
    rng = np.random.default_rng(N)
    lens = np.full(m, 3)
    lens[rng.choice(m, m // 200, replace=False)] = 2000 // mean
    A, B = _rows_of(rng, lens, m), _rows_of(rng, np.full(m, mean), N)
    say("allocation-free m=%d N=%d" % (m, N))
    want, got = _pair(torch_gpu, A, B)
    assert all(np.array_equal(x, y) for x, y in zip(want, got))
    with aires.tile_plan(aires.to_device(A), aires.to_device(B), 0) as plan:
        cap = len(want[1])
        rp = torch_gpu.empty(m + 1, dtype=torch_gpu.int64, device="cuda")
        col = torch_gpu.empty(cap, dtype=torch_gpu.int32, device="cuda")
        val = torch_gpu.empty(cap, dtype=torch_gpu.float32, device="cuda")
        assert aires.spgemm_noalloc(plan, rp, col, val) == cap
        torch_gpu.cuda.synchronize()
        assert aires.plan_stats(plan)["numeric_launches"] == 2
