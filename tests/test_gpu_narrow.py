"""GPU parity of narrow products (N <= 8192) that read B's rows as presence
bitmaps and fixed slots, against the oracle and against the general kernels
(the same plan under a budget that leaves no room for bitmaps and slots)."""
import numpy as np
import pytest

import oracle
import workloads
from workloads import CSR

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch


def csr_of_lengths(rng, lens, ncols, ints):
    lens = np.minimum(np.asarray(lens), ncols)
    rp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = [np.sort(rng.choice(ncols, L, replace=False)) for L in lens]
    col = np.concatenate(col).astype(np.int32) if len(col) else np.zeros(0, np.int32)
    val = rng.integers(-3, 4, len(col)) if ints else rng.uniform(-1, 1, len(col))
    return CSR(len(lens), ncols, rp, col, val.astype(np.float32))


def operands(rng, N, mean, K=700, ints=True):
    """B: rows around `mean` entries, some empty, some far longer than a slot.
    A: row lengths around a step (8 ... 32 entries), a window (128), the
    symbolic phase's parts (1024, 2048) and single entries."""
    lb = np.clip(rng.poisson(mean, K), 0, N)
    lb[rng.choice(K, K // 20, replace=False)] = 0
    lb[rng.choice(K, 5, replace=False)] = N
    B = csr_of_lengths(rng, lb, N, ints)
    # K columns only, so longer rows of A come from a taller B
    la = np.concatenate([np.array([0, 1, 1, 2, 3, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 130, 255,
                                   256, 257, 400, K, 1, 0, 1]), rng.integers(0, 60, 150), np.ones(40, int)])
    return csr_of_lengths(rng, la, K, ints), B


def run(aires, torch, A, B, rp64=(False, False), **kw):
    def dev(M, wide):
        return aires.to_device(CSR(M.nrows, M.ncols, M.rp.astype(np.int64 if wide else np.int32), M.col, M.val))
    with aires.tile_plan(dev(A, rp64[0]), dev(B, rp64[1]), **kw) as plan:
        C = aires.spgemm(plan)
        torch.cuda.synchronize()
        stats = aires.plan_stats(plan)
    return C.rp.cpu().numpy(), C.col.cpu().numpy(), C.val.cpu().numpy(), stats


WIDTHS = [(1, 1), (31, 3), (32, 5), (33, 6), (64, 6), (65, 10), (127, 12), (128, 13), (129, 14), (200, 16), (250, 25),
          (256, 26), (500, 22), (512, 26), (513, 40), (1000, 50), (1024, 60), (2047, 70), (2048, 100), (2048, 300),
          (2049, 30), (3000, 70), (4096, 60), (4097, 45), (6001, 60), (8192, 40), (8193, 60)]


@pytest.mark.parametrize("N,mean", WIDTHS)
def test_widths_and_slot_sizes(torch_gpu, N, mean):
    """Small integer values: every sum is exact, so C equals the oracle's bit
    for bit whatever the order."""
    import paper_2507_02006_amd as aires
    rng = np.random.default_rng(N * 31 + mean)
    A, B = operands(rng, N, mean)
    ref = oracle.spgemm(A, B)
    print("[gpu-case] narrow N=%d mean=%d products=%d" % (N, mean, ref.products), flush=True)
    for rp64 in ((False, False), (True, False), (False, True), (True, True)):
        rp, col, val, st = run(aires, torch_gpu, A, B, rp64)
        assert st["products"] == ref.products
        assert np.array_equal(rp, ref.rp) and np.array_equal(col, ref.col) and np.array_equal(val, ref.val)
    # rows spread over every kernel: a workgroup each, split over slots, tiles
    for kw in (dict(wave_max_products=60, split_min_products=400), dict(wave_max_products=20, split_min_products=-1),
               dict(wave_max_products=30, split_min_products=90, split_max_rows=3, max_tile_rows=37)):
        rp, col, val, _ = run(aires, torch_gpu, A, B, **kw)
        assert np.array_equal(rp, ref.rp) and np.array_equal(col, ref.col) and np.array_equal(val, ref.val)


def test_long_rows_in_parts(torch_gpu):
    """Rows of A around 1024 entries (one lane group or parts), 2048 and 4096
    (the ends of a part), beside rows that touch empty rows of B only."""
    import paper_2507_02006_amd as aires
    rng = np.random.default_rng(3)
    K, N = 9000, 96
    lb = rng.poisson(9, K)
    lb[:4000] = 0
    B = csr_of_lengths(rng, lb, N, True)
    lens = [1023, 1024, 1025, 2047, 2048, 2049, 4096, 4097, 8999, 9000, 5, 0, 3000]
    A = csr_of_lengths(rng, lens, K, True)
    empty = np.sort(rng.choice(4000, 2500, replace=False)).astype(np.int32)  # P_i = 0 with many entries
    A = CSR(A.nrows + 1, K, np.append(A.rp, A.rp[-1] + len(empty)), np.concatenate([A.col, empty]),
            np.concatenate([A.val, np.ones(len(empty), np.float32)]))
    ref = oracle.spgemm(A, B)
    for kw in ({}, dict(split_min_products=5000), dict(max_tile_rows=3)):
        rp, col, val, st = run(aires, torch_gpu, A, B, **kw)
        assert st["products"] == ref.products
        assert np.array_equal(rp, ref.rp) and np.array_equal(col, ref.col) and np.array_equal(val, ref.val)


class LoggingAllocator:
    """torch-backed allocator that keeps the sizes it handed out and got back."""

    def __init__(self):
        from paper_2507_02006_amd import _binding as B_
        self.inner = B_.TorchAllocator(0)
        self.events, self.size = [], {}
        self._alloc, self._free = B_.ALLOC_FN(self._alloc_cb), B_.FREE_FN(self._free_cb)
        self.struct = B_.Allocator(self._alloc, self._free, None)
        self.take = self.inner.take

    def _alloc_cb(self, ctx, nbytes, stream):
        at = self.inner._alloc_cb(ctx, nbytes, stream)
        self.size[at] = nbytes
        self.events.append(nbytes)
        return at

    def _free_cb(self, ctx, ptr, stream):
        self.events.append(-self.size.pop(ptr, 0))
        self.inner._free_cb(ctx, ptr, stream)


@pytest.mark.parametrize("N,mean,K,m", [(64, 6, 9000, 10400), (500, 22, 6000, 1700), (2048, 100, 2000, 400),
                                        (5000, 50, 2000, 500)])
def test_against_the_general_kernels(torch_gpu, N, mean, K, m):
    """The same product by the general kernels (a hash limit asks for them), with
    no room for bitmaps and slots, with room for the bitmaps alone, and with
    room for both but not for C beside them, so that they are given back: the
    same structure, and values within the bound of two fp32 sums of n terms,
    gamma_n sum |a b| each; infinite and NaN entries reach the same entries of
    C.  The sizes asked of the allocator say which of these it was."""
    import paper_2507_02006_amd as aires
    rng = np.random.default_rng(N)
    lb = np.clip(rng.poisson(mean, K), 0, N)
    lb[rng.choice(K, K // 20, replace=False)] = 0
    lb[rng.choice(K, 5, replace=False)] = N
    B = csr_of_lengths(rng, lb, N, False)
    la = np.concatenate([np.array([0, 1, 1, 2, 7, 8, 9, 31, 32, 33, 63, 64, 65, 127, 128, 129, 257, 400, K, 1, 0, 1]),
                         rng.integers(0, 60, m), np.ones(40, int)])
    A = csr_of_lengths(rng, la, K, False)
    A.val[rng.choice(len(A.val), 3, replace=False)] = [np.inf, -np.inf, np.nan]
    dA, dB = aires.to_device(A), aires.to_device(B)
    inputs = A.nbytes() + B.nbytes()

    def go(budget, **kw):
        log = LoggingAllocator()
        with aires.tile_plan(dA, dB, budget, allocator=log, split_min_products=-1, **kw) as plan:
            planned = aires.plan_info(plan).peak_bytes
            C = aires.spgemm(plan)
            torch_gpu.cuda.synchronize()
        return C.rp.cpu().numpy(), C.col.cpu().numpy(), C.val.cpu().numpy(), log, planned

    *ref, log, planned = go(0)
    *gen, glog, _ = go(0, hash_max_products=4096)
    both = log.inner.peak - glog.inner.peak
    bits = 256 * (-(-4 * narrow_words(N) * K // 256) + -(-4 * narrow_words(N) * A.nrows // 256))
    assert both >= bits and both in log.events and both not in glog.events
    compare(A, B, *gen, *ref)
    least = inputs + glog.inner.peak  # holds C and the general path's workspace
    print("[gpu-case] general path N=%d: C %d, bitmaps and slots %d bytes" % (N, 8 * len(ref[1]), both), flush=True)
    # no room for the bitmaps
    assert least - planned < bits
    *got, log, _ = go(max(planned + 1, least))
    assert log.inner.peak == glog.inner.peak
    compare(A, B, *got, *ref)
    # room for them, but not for C beside them
    budget = max(planned + both, least)
    assert budget < least + both
    *got, log, _ = go(budget)
    assert both in log.events and log.events.index(-both) < log.events.index(4 * len(ref[1]))
    compare(A, B, *got, *ref)
    if both > bits + 4096:  # slots too: room for the bitmaps alone, and C beside them
        budget = planned + both - 1
        assert least + bits + 65536 <= budget
        *got, log, _ = go(budget)
        taken = log.inner.peak - glog.inner.peak
        assert bits <= taken < bits + 65536
        compare(A, B, *got, *ref)


def narrow_words(N):
    words = 4
    while 32 * words < N:
        words *= 2
    return words


def compare(A, B, rp, col, val, probe_rp, probe_col, probe_val):
    assert np.array_equal(rp, probe_rp) and np.array_equal(col, probe_col)
    fin = np.isfinite(val)
    assert np.array_equal(fin, np.isfinite(probe_val))
    assert np.array_equal(np.isnan(val), np.isnan(probe_val))
    inf = ~fin & ~np.isnan(val)
    assert np.array_equal(val[inf], probe_val[inf])
    Aabs = CSR(A.nrows, A.ncols, A.rp, A.col, np.abs(np.nan_to_num(A.val, posinf=0, neginf=0)))
    mag = oracle.spgemm(Aabs, CSR(B.nrows, B.ncols, B.rp, B.col, np.abs(B.val)))
    n = np.repeat(np.diff(A.rp), np.diff(rp))
    bound = 2 * (n + 2) * 2.0 ** -24 * mag.val
    assert np.all(np.abs(val[fin].astype(np.float64) - probe_val[fin]) <= bound[fin] + 1e-30)


@pytest.mark.parametrize("N", [2049, 5000, 12001, 16384])
def test_wide_dense_rows_split_in_parts(torch_gpu, N):
    """Products of 2049 to 16384 columns whose heavy rows are cut into parts of
    16384 products (one to several), with slots for all of them, for two of
    them and for none, in tiles, and with the bitmaps of B off (a hash limit is
    asked for) and on; integer values, so exact."""
    import paper_2507_02006_amd as aires
    rng = np.random.default_rng(N)
    K = 1500
    B = csr_of_lengths(rng, np.clip(rng.poisson(45, K), 0, N), N, True)
    lens = [K, 800, 400, 365, 363, 200, 90, 40, 10, 1, 0] + [5] * 60 + [1200, 700]
    A = csr_of_lengths(rng, lens, K, True)
    ref = oracle.spgemm(A, B)
    print("[gpu-case] wide split N=%d" % N, flush=True)
    base = dict(split_min_products=12000)
    for kw in (base, dict(base, split_max_rows=2), dict(split_min_products=-1), dict(base, max_tile_rows=30),
               dict(base, hash_max_products=4096), dict(base, hash_max_products=4096, max_tile_rows=30)):
        rp, col, val, st = run(aires, torch_gpu, A, B, **kw)
        assert st["products"] == ref.products
        assert np.array_equal(rp, ref.rp) and np.array_equal(col, ref.col) and np.array_equal(val, ref.val)


@pytest.mark.parametrize("N,mean,least", [(64, 6, 0.9), (512, 25, 2.0), (5000, 60, 2.5)])
def test_bitmaps_of_b_only_for_enough_entries_of_a(torch_gpu, N, mean, least):
    """Bitmaps (and slots) are written for every row of B, so a few rows of A
    against a tall B must not ask for them: the call's device memory, counted
    at the allocator, stays below what they take; from `least` entries of A per
    row of B on they are there.  Integer values, so both are exact."""
    import paper_2507_02006_amd as aires
    from paper_2507_02006_amd import _binding as B_
    rng = np.random.default_rng(N)
    K = 60000
    B = csr_of_lengths(rng, np.clip(rng.poisson(mean, K), 1, N), N, True)
    dB = aires.to_device(B)
    words = narrow_words(N)
    for per_row, expect in ((0.01, False), (0.9 * least, False), (1.1 * least, True)):
        A = csr_of_lengths(rng, np.full(int(K * per_row / 60), 60), K, True)
        ref = oracle.spgemm(A, B)
        log = B_.TorchAllocator(0)
        with aires.tile_plan(aires.to_device(A), dB, 0, allocator=log, split_min_products=-1) as plan:
            C = aires.spgemm(plan)
            torch_gpu.cuda.synchronize()
        extra = log.peak - 8 * ref.nnz  # without C's entries
        print("[gpu-case] bitmaps N=%d nnz(A)/K=%.2f: %d bytes beside C" % (N, A.nnz / K, extra), flush=True)
        assert (extra >= 4 * words * K) == expect
        assert np.array_equal(C.rp.cpu().numpy(), ref.rp) and np.array_equal(C.col.cpu().numpy(), ref.col)
        assert np.array_equal(C.val.cpu().numpy(), ref.val)


def test_b_of_two_to_the_thirty_rows(torch_gpu):
    """As many rows of B as one launch that writes their bitmaps could not
    hold: a quarter of them with one entry each, A with enough entries that
    bitmaps would pay.  Counts, so exact."""
    import paper_2507_02006_amd as aires
    torch = torch_gpu
    K, N, m, per = 1 << 30, 64, 4096, 27001
    have = K // 4
    brp = torch.arange(K + 1, dtype=torch.int32, device="cuda").clamp_(max=have)
    bcol = torch.arange(have, dtype=torch.int32, device="cuda") % N
    bval = torch.ones(have, device="cuda")
    step = K // per
    acol = (torch.arange(per, dtype=torch.int32, device="cuda") * step)[None, :] + (
        torch.arange(m, dtype=torch.int32, device="cuda") * 7)[:, None]  # below step
    assert (per - 1) * step + 7 * (m - 1) < K and 7 * (m - 1) < step
    arp = torch.arange(m + 1, dtype=torch.int64, device="cuda") * per
    A = (m, K, arp, acol.reshape(-1).contiguous(), torch.ones(m * per, device="cuda"))
    print("[gpu-case] B of 2^30 rows", flush=True)
    with aires.tile_plan(A, (K, N, brp, bcol, bval)) as plan:
        C = aires.spgemm(plan)
        torch.cuda.synchronize()
    k = acol.long()
    key = (torch.arange(m, device="cuda")[:, None] * N + k % N)[k < have]
    count = torch.bincount(key, minlength=m * N).reshape(m, N)
    lens = (count > 0).sum(1)
    assert torch.equal(C.rp[1:] - C.rp[:-1], lens)
    assert torch.equal(C.col.long(), count.nonzero()[:, 1])
    assert torch.equal(C.val, count[count > 0].float())
    del C, A, brp, bcol, bval, acol, k, key
    torch.cuda.empty_cache()


@pytest.mark.parametrize("N,mean,m,length,expect", [(200, 20, 8, 1500, True), (200, 20, 8, 900, False), (64, 6, 2, 9000, True),
                                                    (8000, 120, 1, 20000, True), (8000, 120, 30, 400, False),
                                                    (4000, 100, 1, 20000, False)])
def test_bitmaps_of_b_for_few_long_rows_of_a(torch_gpu, N, mean, m, length, expect):
    """Few long rows of A take bitmaps (and slots) of B from far fewer entries
    on: a row is one workgroup's work otherwise.  The device memory beside C
    says which path ran; integer values, so both are exact."""
    import paper_2507_02006_amd as aires
    from paper_2507_02006_amd import _binding as B_
    rng = np.random.default_rng(N + m)
    K = 60000
    B = csr_of_lengths(rng, np.clip(rng.poisson(mean, K), 1, N), N, True)
    A = csr_of_lengths(rng, np.full(m, length), K, True)
    words = narrow_words(N)
    ref = oracle.spgemm(A, B)
    log = B_.TorchAllocator(0)
    with aires.tile_plan(aires.to_device(A), aires.to_device(B), 0, allocator=log, split_max_rows=1) as plan:
        C = aires.spgemm(plan)
        torch_gpu.cuda.synchronize()
    extra = log.peak - 8 * ref.nnz
    print("[gpu-case] long rows N=%d m=%d length=%d: %d bytes beside C" % (N, m, length, extra), flush=True)
    assert (extra >= 4 * words * K) == expect
    assert np.array_equal(C.rp.cpu().numpy(), ref.rp) and np.array_equal(C.col.cpu().numpy(), ref.col)
    assert np.array_equal(C.val.cpu().numpy(), ref.val)


@pytest.mark.parametrize("N", [1024, 8192])
def test_long_rows_of_b_do_not_hold_up_the_bitmaps(torch_gpu, N):
    """Rows of B with an entry in every column, which A does not touch: writing
    their bitmaps (and slots) costs a call at most 75 us (8192 entries read 16
    at a time took 120)."""
    import paper_2507_02006_amd as aires
    torch = torch_gpu
    rng = np.random.default_rng(N)
    K = 20000
    lens = rng.poisson(60, K)
    full = np.arange(7, K, 500)
    A = csr_of_lengths(rng, np.full(8000, 16), K - len(full), True)
    A = CSR(A.nrows, K, A.rp, np.setdiff1d(np.arange(K), full)[A.col].astype(np.int32), A.val)
    best = {}
    for name in ("short", "long"):
        if name == "long":
            lens[full] = N
        B = csr_of_lengths(np.random.default_rng(1), lens, N, True)
        dA, dB = aires.to_device(A), aires.to_device(B)
        best[name] = float("inf")
        for _ in range(15):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            torch.cuda.synchronize()
            a.record()
            with aires.tile_plan(dA, dB) as plan:
                aires.spgemm(plan)
            b.record()
            b.synchronize()
            best[name] = min(best[name], a.elapsed_time(b) * 1e3)
    print("[gpu-case] full rows of B, N=%d: %s us" % (N, best), flush=True)
    assert best["long"] <= best["short"] + 75.0


@pytest.mark.parametrize("m", [5000, 20000])
def test_phase_times_of_the_bitmap_path(torch_gpu, m):
    """The times of a call with bitmaps: products are counted in the symbolic
    pass (no analysis), binning is a phase of its own, and the scan too where
    the rows are not few."""
    import paper_2507_02006_amd as aires
    rng = np.random.default_rng(m)
    A, B = csr_of_lengths(rng, [9] * m, 4000, True), csr_of_lengths(rng, [12] * 4000, 128, True)
    with aires.tile_plan(aires.to_device(A), aires.to_device(B), timing=True) as plan:
        aires.spgemm(plan)
        torch_gpu.cuda.synchronize()
        st, tile = aires.plan_stats(plan), aires.plan_tile_stats(plan, 0)
    for x in (st, tile):
        assert x["analyze_ms"] == 0.0 and x["symbolic_ms"] > 0.0 and x["numeric_ms"] > 0.0
        assert x["bin_ms"] > 0.0 and (x["scan_ms"] > 0.0) == (m > 8192)
