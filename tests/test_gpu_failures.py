"""Calls that fail leave nothing behind: an allocation that fails at any point
of a product is reported, and the same thread's next product, on another
stream and while the failed one's kernels are still queued, is right."""
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
            return None if self.calls - 1 == n else L._torch_alloc(nbytes, ctx, stream)

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
