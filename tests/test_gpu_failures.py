"""Allocations that fail.  One at any point of a product is reported and leaves
nothing behind: the same thread's next product, on another stream and while
the failed one's kernels are still queued, is right.  The backward goes on
without its optional scratch; the forms that it then takes, and others for
sizes that few products have, give the same values."""
import numpy as np
import pytest

import synthetic as S

pytestmark = pytest.mark.gpu


class FailingAlloc:
    """The binding's allocator with the n-th allocation failing (n from 0)."""

    def __init__(self, L, n):
        self.n, self.calls = n, 0

        def alloc(nbytes, ctx, stream):
            self.calls += 1
            return None if self.calls - 1 == self.n else L._torch_alloc(nbytes, ctx, stream)

        self.cb = L._ALLOC_T(alloc)


@pytest.mark.parametrize("case", ["short", "merge", "windows"])
def test_product_after_a_failed_allocation(case, monkeypatch):
    import torch
    from paper_1504_05022_amd import lib as L
    if case == "short":
        ci = np.sort((np.arange(5000)[:, None] + [0, 7, 100, 1000]) % 5000, axis=1)
        A = S.Csr(5000, 5000, np.arange(0, 20001, 4, dtype=np.int32),
                  ci.ravel().astype(np.int32), np.random.default_rng(1).standard_normal(20000))
        B = A
    elif case == "merge":
        A, _ = S.config2(n=5000, cap=1500)
        B = A
    else:
        A, B = S.crafted_rows([600, 3000, 40000, 513, 20] * 4, n=1500)
    dA, dB = L.CsrMatrix.from_host(A), L.CsrMatrix.from_host(B)
    ref = L.spgemm(dA, dB).to_host()
    other, _ = S.config2(n=3000, cap=900)
    dO = L.CsrMatrix.from_host(other)
    ref_o = L.spgemm(dO, dO).to_host()
    busy = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    good = L._alloc_cb
    n = 0
    while True:
        print("case: %s, allocation %d fails" % (case, n), flush=True)
        fa = FailingAlloc(L, n)
        failed = False
        with torch.cuda.stream(s1):
            for _ in range(2):
                busy @ busy  # holds the stream: what the call queues runs late
            monkeypatch.setattr(L, "_alloc_cb", fa.cb)
            try:
                L.spgemm(dA, dB)
            except L.SpgemmError as e:
                assert e.name == "ENOMEM"
                failed = True
            monkeypatch.setattr(L, "_alloc_cb", good)
        with torch.cuda.stream(s2):
            got = L.spgemm(dO, dO)
            s2.synchronize()
        for x, y in zip(got.to_host()[2:], ref_o[2:]):
            assert np.array_equal(x, y)
        torch.cuda.synchronize()
        if not failed:
            assert fa.calls == n  # every allocation of the call has failed once
            break
        n += 1
    assert n >= 5  # analysis, C~, and C's three arrays
    for x, y in zip(L.spgemm(dA, dB).to_host()[2:], ref[2:]):
        assert np.array_equal(x, y)


def _csr(rows, cols, lens, rng, dtype=np.float64):
    rp = np.r_[0, np.cumsum(lens)].astype(np.int32)
    ci = np.concatenate([np.sort(rng.choice(cols, n, replace=False)) for n in lens])
    return S.Csr(rows, cols, rp, ci.astype(np.int32), rng.standard_normal(ci.size).astype(dtype))


@pytest.mark.parametrize("n", [0, 1, 2])
def test_backward_without_its_scratch(n):
    """The temporary space of the transposed pattern, the pattern beside it and
    the staged products refused in turn: the backward goes on without, to the
    same values, and again on the same plan."""
    import torch
    from paper_1504_05022_amd import lib as L
    rng = np.random.default_rng(8)
    A = L.CsrMatrix.from_host(_csr(3000, 700, rng.integers(0, 20, 3000), rng))
    B = L.CsrMatrix.from_host(_csr(700, 900, rng.integers(0, 30, 700), rng))
    plan = L.Plan(A, B)
    C = plan.compute()
    dC = torch.randn(C.nnz, device="cuda", dtype=torch.float64)
    ref = plan.backward(C, dC)
    fa = FailingAlloc(L, -1)
    good, L._alloc_cb = L._alloc_cb, fa.cb
    try:
        plan = L.Plan(A, B)
    finally:
        L._alloc_cb = good
    C = plan.compute()
    fa.n, fa.calls = n, 0
    for r in range(2):
        print("case: allocation %d of the backward fails, call %d" % (n, r), flush=True)
        for got, want in zip(plan.backward(C, dC), ref):
            assert torch.equal(got, want)
    assert fa.calls > n
    plan.close()


@pytest.mark.parametrize("k", [(1 << 21) - 1, 1 << 21, (1 << 21) + 1])
def test_backward_around_the_widest_partition(k):
    """A's columns around the number up to which its transposed pattern is
    partitioned: dB against sequential sums."""
    import torch
    from paper_1504_05022_amd import CsrMatrix, Plan
    rng = np.random.default_rng(k)
    cols = np.sort(rng.choice(k, 500, replace=False))
    cols[[0, -1]] = 0, k - 1
    A = _csr(400, 500, rng.integers(0, 40, 400), rng)
    A = S.Csr(400, k, A.row_ptr, cols[A.col_idx].astype(np.int32), A.val)
    brp = np.zeros(k + 1, np.int64)
    brp[cols + 1] = 1
    B = S.Csr(k, 3, np.cumsum(brp).astype(np.int32), (np.arange(500) % 3).astype(np.int32),
              rng.standard_normal(500))
    print("case: k %d" % k, flush=True)
    plan = Plan(CsrMatrix.from_host(A), CsrMatrix.from_host(B))
    C = plan.compute()
    dc = rng.standard_normal(C.nnz)
    _, gB = plan.backward(C, torch.from_numpy(dc).cuda(), want_a=False)
    _, _, crp, cci, _ = C.to_host()
    dense = np.zeros((400, 3))
    dense[np.repeat(np.arange(400), np.diff(crp)), cci] = dc
    at = np.searchsorted(cols, A.col_idx)
    ref = np.zeros(500)
    np.add.at(ref, at, A.val * dense[np.repeat(np.arange(400), np.diff(A.row_ptr)), at % 3])
    assert np.array_equal(gB.cpu().numpy(), ref)


def test_dense_windows_of_many_long_rows():
    """More long rows than one work-group can add up the planning sums of
    (262144), by thresholds that make every row long."""
    from test_gpu_parity import check
    rng = np.random.default_rng(2)
    m = 262144 + 300
    A = _csr(64, 64, np.full(64, 3), rng, np.float32)
    ci = np.tile(A.col_idx, m // 64 + 1)[:3 * m]
    A = S.Csr(m, 64, np.arange(0, 3 * m + 1, 3, dtype=np.int32), ci,
              rng.standard_normal(3 * m).astype(np.float32))
    B = _csr(64, 100, np.full(64, 4), rng, np.float32)
    check(A, B, bin_edges=(1, 2, 3, 4, 5))
