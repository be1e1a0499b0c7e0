"""Kernels at the sizes where they can go wrong: edges of tiles, windows and
chunks, remainders, empty rows.  Tolerances are error bounds of the sums."""
import numpy as np
import pytest

import oracle
import synthetic as S

pytestmark = pytest.mark.gpu


def _ragged(rng, rows, lengths, cols, dtype):
    """Rows of the given lengths (in that order), distinct uniform columns."""
    rp = np.zeros(rows + 1, np.int32)
    rp[1:] = np.cumsum(lengths)
    ci = np.concatenate([np.sort(rng.choice(cols, n, replace=False)) for n in lengths]
                        + [np.zeros(0, np.int64)])
    return S.Csr(rows, cols, rp, ci.astype(np.int32), rng.standard_normal(ci.size).astype(dtype))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("n", [40, 8192, 8193])
def test_backward_ragged_rows(dtype, n):
    """Rows of B around blocks of 64 products and windows of 2048 of them,
    rows of A around batches of 64 and chunks of 128 entries, B up to the
    widest bitmap and one column beyond."""
    import torch
    from paper_1504_05022_amd import CsrMatrix, Plan
    rng = np.random.default_rng(5)
    lens = [0, 0, 1, 2, 31, 63, 64, 65, 127, 128, 129, 2047, 2048, 2049, 5000]
    lens = [min(x, n) for x in lens] * 10
    rng.shuffle(lens)
    k = len(lens)
    B = _ragged(rng, k, lens, n, dtype)
    A = _ragged(rng, 15, [0, 1, 63, 64, 65, 0, 127, 128, 129, 130, 0, 0, 3, 2, 0], k, dtype)
    print("case: n %d %s products of %d entries" % (n, np.dtype(dtype), A.nnz), flush=True)
    dA, dB = CsrMatrix.from_host(A), CsrMatrix.from_host(B)
    plan = Plan(dA, dB)
    C = plan.compute()
    dc = rng.standard_normal(C.nnz).astype(dtype)
    gA, gB = plan.backward(C, torch.from_numpy(dc).cuda())
    torch.cuda.synchronize()
    _, _, rp, ci, _ = C.to_host()

    def grads(f):
        x, y = A.astype(np.float64), B.astype(np.float64)
        x.val, y.val = f(x.val), f(y.val)
        return oracle.grad(x.as_tuple(), y.as_tuple(), rp.astype(np.int64), ci,
                           f(dc.astype(np.float64)))

    refs, mags = grads(lambda v: v), grads(np.abs)
    # a sum of t rounded products is off by at most (t + 1) eps times the
    # sum of their magnitudes, in whatever order it is added
    eps = np.finfo(dtype).eps
    terms = (np.array(lens)[A.col_idx], np.bincount(A.col_idx, minlength=k).repeat(lens))
    for got, ref, mag, t in zip((gA, gB), refs, mags, terms):
        assert np.all(np.abs(got.cpu().numpy() - ref) <= (t + 2) * eps * mag)


@pytest.mark.parametrize("n", [8192, 8193])
def test_backward_full_chunks(n):
    """Enough entries of A for chunks of 128 and 64 of them per wavefront (a
    smaller A takes fewer), with windows of 2048 products inside them."""
    import torch
    from paper_1504_05022_amd import CsrMatrix, Plan
    rng = np.random.default_rng(6)
    k, m = 500, 2700
    lens = [int(x) for x in np.r_[rng.integers(0, 60, k - 12), [2047, 2048, 2049, 64] * 3]]
    B = _ragged(rng, k, lens, n, np.float64)
    A = _ragged(rng, m, rng.integers(0, 200, m), k, np.float64)
    A = S.Csr(m, k, A.row_ptr, A.col_idx, np.abs(A.val))
    assert A.nnz > 2048 * 128
    print("case: n %d products of %d entries" % (n, A.nnz), flush=True)
    plan = Plan(CsrMatrix.from_host(A), CsrMatrix.from_host(B))
    C = plan.compute()
    dc = rng.standard_normal(C.nnz)
    gA, gB = plan.backward(C, torch.from_numpy(dc).cuda())
    _, _, rp, ci, _ = C.to_host()
    args = (rp.astype(np.int64), ci)
    refs = oracle.grad(A.as_tuple(), B.as_tuple(), *args, dc)
    absB = S.Csr(k, n, B.row_ptr, B.col_idx, np.abs(B.val))
    mags = oracle.grad(A.as_tuple(), absB.as_tuple(), *args, np.abs(dc))
    eps = np.finfo(np.float64).eps  # a sum of t rounded products, in any order
    terms = (np.array(lens)[A.col_idx], np.bincount(A.col_idx, minlength=k).repeat(lens))
    for got, ref, mag, t in zip((gA, gB), refs, mags, terms):
        assert np.all(np.abs(got.cpu().numpy() - ref) <= (t + 2) * eps * mag)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("col_range", [None, 60])
def test_short_rows_around_network_sizes(dtype, col_range):
    """Row sizes on both sides of every number of products per lane that the
    short-row kernels choose (5, 6, 7, 8 and 10, 12, 16 times the lanes per
    row), alone in a wavefront and beside rows of other sizes, with few and
    with many equal columns, and with runs of B of one to many products:
    bit-exact against the sequential sums."""
    from test_gpu_parity import check
    sizes = [g * k + d for g in (16, 32, 64) for k in (4, 5, 6, 7, 8) for d in (-1, 0, 1)]
    sizes += [64 * k + d for k in (10, 12, 16) for d in (-1, 0, 1)]
    sizes = [s for s in sorted(set(sizes)) if s <= 1024]
    targets = sizes * 2 + [s for s in sizes for _ in range(4)]
    A, B = S.crafted_rows(targets, col_range=col_range, empty_refs=3, dtype=dtype)
    check(A, B, long_path=1, bin_edges=(32, 64, 128, 256, 1024))


@pytest.mark.parametrize("m", [0, 1, 4096, 4097, 32768, 131071, 131072, 262144, 262145])
def test_row_counts_around_binning_and_copy_sizes(m):
    """Row counts at the limits of the one-work-group binning, of its rows per
    thread and of the copy's rows per wavefront; empty rows, rows of one to a
    few hundred products and a long row among them."""
    from test_gpu_parity import check
    rng = np.random.default_rng(m)
    B = _ragged(rng, 64, [0, 1, 2, 40] * 16, 5000, np.float64)
    lens = np.arange(m) % 5
    lens[-3:] = min(m, 60)
    A = _ragged(rng, m, lens, 64, np.float64)
    check(A, B)


@pytest.mark.parametrize("k", [1, 2, 1024, 1025, 4096])
def test_db_over_transposed_pattern_parts(k):
    """Columns of A from one to several groups of them, entries around tiles
    of 8192 and wavefronts of 2048, a column in every row, empty columns:
    dB, whose sums run in the order of A's rows, equals sequential sums."""
    import torch
    from paper_1504_05022_amd import CsrMatrix, Plan
    rng = np.random.default_rng(k)
    for rows in (1, 2047, 8191, 8193, 20001):
        lens = np.minimum(rng.integers(0, 4, rows), k)
        A = _ragged(rng, rows, lens, k, np.float64)
        # every row also holds column 0
        entries = [np.unique(np.r_[0, A.col_idx[a:b]])
                   for a, b in zip(A.row_ptr[:-1], A.row_ptr[1:])]
        rp = np.r_[0, np.cumsum([x.size for x in entries])].astype(np.int32)
        ci = np.concatenate(entries).astype(np.int32)
        A = S.Csr(rows, k, rp, ci, rng.standard_normal(ci.size))
        B = S.Csr(k, 3, np.arange(k + 1, dtype=np.int32), (np.arange(k) % 3).astype(np.int32),
                  rng.standard_normal(k))
        print("case: %d x %d, %d entries" % (rows, k, ci.size), flush=True)
        dA, dB = CsrMatrix.from_host(A), CsrMatrix.from_host(B)
        plan = Plan(dA, dB)
        C = plan.compute()
        dc = rng.standard_normal(C.nnz)
        _, gB = plan.backward(C, torch.from_numpy(dc).cuda(), want_a=False)
        _, _, crp, cci, _ = C.to_host()
        dense = np.zeros((rows, 3))
        dense[np.repeat(np.arange(rows), np.diff(crp)), cci] = dc
        prod = A.val * dense[np.repeat(np.arange(rows), np.diff(rp)), ci % 3]
        ref = np.zeros(k)
        np.add.at(ref, ci, prod)  # in the order of the entries
        assert np.array_equal(gB.cpu().numpy(), ref)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("most", [16, 17, 32, 33, 64, 65, 200])
def test_dense_windows_by_b_row_length(dtype, most):
    """Long rows of a narrow product whose rows of B are all at most 16, at
    most 32 or longer (alone, two and four to a wavefront), with equal columns
    in neighbouring rows, empty rows and partly filled batches; one row above
    the size that is cut into product ranges."""
    from test_gpu_parity import check
    rng = np.random.default_rng(most)
    n = 256
    lens = np.r_[most, rng.integers(0, most + 1, 199)]
    B = _ragged(rng, 200, lens, n, dtype)
    deg = [d for d in (5, 63, 64, 65, 127, 130, 199, 200) for _ in range(6)]
    A = _ragged(rng, len(deg), deg, 200, dtype)
    check(A, B, exact=bool(np.sum(lens) <= 16384))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("rare", [33, 64, 65, 200])
def test_dense_windows_with_a_rare_long_row(dtype, rare):
    """Rows of B of at most 16 entries but for one in 200: the kernel for short
    rows, in whose batches the long one is met alone."""
    from test_gpu_parity import check
    rng = np.random.default_rng(rare)
    lens = np.r_[rng.integers(8, 17, 100), rare, rng.integers(8, 17, 99)]
    B = _ragged(rng, 200, lens, 256, dtype)
    deg = [d for d in (63, 64, 65, 130, 199, 200) for _ in range(6)]
    A = _ragged(rng, len(deg), deg, 200, dtype)
    check(A, B)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("u", [(1025, 600), (3000, 1025, 4000), (40000, 4100, 520, 3000)])
def test_long_rows_in_few_columns(dtype, u):
    """Cut rows of C whose products share one range of columns: streams above
    a wavefront's 1024 entries, up to and above a work-group's 4096, beside
    rows that have none."""
    from test_gpu_parity import check
    rng = np.random.default_rng(len(u))
    n, width = 20000, 20
    deg = [x // width for x in u] + [3]
    k = max(deg)
    lens = [width] * k
    B = _ragged(rng, k, lens, 48, dtype)
    B = S.Csr(k, n, B.row_ptr, B.col_idx + 77, B.val)
    A = _ragged(rng, len(deg), deg, k, dtype)
    check(A, B)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_backward_wide_rows_around_samples(dtype):
    """C wider than a bitmap, its rows around the 1024 columns that are sampled
    for the searches and the strides above, short and long rows and empty ones
    in one batch of entries; more rows than lanes in a chunk; very few
    products against a long row of C."""
    import torch
    from paper_1504_05022_amd import CsrMatrix, Plan
    rng = np.random.default_rng(9)
    n = 40000
    lens = [0, 1, 1, 2, 500, 1023, 1024, 1025, 2048, 2049, 5000, 0] + [1] * 200
    k = len(lens)
    B = _ragged(rng, k, lens, n, dtype)
    rows = [[4], [5], [6], [7], [8], [9], [10], [], [1, 2, 10], [0, 11], list(range(12)),
            list(range(12, k))] + [[12 + x] for x in range(150)] + [[]] * 80 + [[3, 10, 20, 30]]
    rp = np.r_[0, np.cumsum([len(r) for r in rows])].astype(np.int32)
    ci = np.concatenate([np.array(r, np.int32) for r in rows])
    A = S.Csr(len(rows), k, rp, ci.astype(np.int32), rng.standard_normal(ci.size).astype(dtype))
    print("case: %s products of %d entries" % (np.dtype(dtype), A.nnz), flush=True)
    plan = Plan(CsrMatrix.from_host(A), CsrMatrix.from_host(B))
    C = plan.compute()
    dc = rng.standard_normal(C.nnz).astype(dtype)
    gA, gB = plan.backward(C, torch.from_numpy(dc).cuda())
    _, _, crp, cci, _ = C.to_host()

    def grads(f):
        x, y = A.astype(np.float64), B.astype(np.float64)
        x.val, y.val = f(x.val), f(y.val)
        return oracle.grad(x.as_tuple(), y.as_tuple(), crp.astype(np.int64), cci,
                           f(dc.astype(np.float64)))

    refs, mags = grads(lambda v: v), grads(np.abs)
    eps = np.finfo(dtype).eps  # a sum of t rounded products, in any order
    terms = (np.array(lens)[A.col_idx], np.bincount(A.col_idx, minlength=k).repeat(lens))
    for got, ref, mag, t in zip((gA, gB), refs, mags, terms):
        assert np.all(np.abs(got.cpu().numpy() - ref) <= (t + 2) * eps * mag)


def test_training_steps_give_their_memory_back():
    """The plan and the matrices of a differentiable product are released with
    its last tensor, without Python's cycle collector."""
    import gc
    import torch
    from paper_1504_05022_amd import CsrMatrix, matmul
    rng = np.random.default_rng(3)
    A = CsrMatrix.from_host(_ragged(rng, 300, [20] * 300, 300, np.float64))
    A.val.requires_grad_(True)

    def step():
        C = matmul(A, A)
        torch.autograd.grad(C.val.sum(), A.val)

    step()
    gc.collect()
    gc.disable()
    try:
        base = torch.cuda.memory_allocated()
        for _ in range(3):
            step()
        assert torch.cuda.memory_allocated() == base
    finally:
        gc.enable()


@pytest.mark.parametrize("count", [1, 580, 680])
def test_one_shot_batch_of_many_problems(count):
    """One-shot batches up to and beyond the counts that fit the pinned area,
    with an empty problem and one that goes through the plain path."""
    from paper_1504_05022_amd import CsrMatrix, batch_multiply
    rng = np.random.default_rng(count)
    pairs = []
    for p in range(count):
        n = 1 + p % 4
        lens = np.zeros(n, int) if p == 5 else rng.integers(0, n + 1, n)
        pairs.append((_ragged(rng, n, lens, n, np.float64), _ragged(rng, n, lens, n, np.float64)))
    wide = _ragged(rng, 60, [40] * 60, 60, np.float32)  # 1600 products per row
    pairs.insert(count // 2, (wide, wide))
    print("case: %d problems" % len(pairs), flush=True)
    out = batch_multiply([(CsrMatrix.from_host(a), CsrMatrix.from_host(b)) for a, b in pairs])
    for C, (a, b) in zip(out, pairs):
        _, _, rp, ci, v = C.to_host()
        ref = oracle.spgemm(a.astype(np.float64).as_tuple(), b.astype(np.float64).as_tuple())
        assert np.array_equal(rp, ref.row_ptr) and np.array_equal(ci, ref.col_idx)
        # a sum of t rounded products: t eps of the sum of their magnitudes
        scale = 40 * np.finfo(v.dtype).eps
        mag = oracle.spgemm(a.astype(np.float64).as_tuple()[:4] + (np.abs(a.val.astype(float)),),
                            b.astype(np.float64).as_tuple()[:4] + (np.abs(b.val.astype(float)),))
        assert np.all(np.abs(v - ref.val) <= scale * mag.val)


def test_products_from_threads_on_their_streams():
    """Plans of several threads, each on a stream of its own, share the second
    streams and wait for their own records: same results as one by one."""
    import threading
    import torch
    from paper_1504_05022_amd import CsrMatrix, Plan, spgemm
    cases = [S.config2(n=n, cap=1500)[0] for n in (3000, 5000, 7000)]
    mats = [CsrMatrix.from_host(A) for A in cases]
    refs = [spgemm(M, M).to_host() for M in mats]
    torch.cuda.synchronize()
    errors = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for r in range(8):
                    M, ref = mats[(k + r) % 3], refs[(k + r) % 3]
                    plan = Plan(M, M)
                    for _ in range(2):
                        C = plan.compute()
                        torch.cuda.current_stream().synchronize()
                        for got, want in zip(C.to_host()[2:], ref[2:]):
                            assert np.array_equal(got, want)
        except BaseException as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


@pytest.mark.parametrize("m", [4000, 70000, 300000])
def test_plan_computed_on_another_stream(m):
    """A plan is whole when it is returned: computed at once on a stream that
    nothing orders behind the one it was analysed on, by each form of the
    binning (one work-group, one and four rows per thread)."""
    import torch
    from paper_1504_05022_amd import CsrMatrix, Plan, spgemm
    rng = np.random.default_rng(m)
    B = CsrMatrix.from_host(_ragged(rng, 64, [0, 1, 2, 40] * 16, 5000, np.float64))
    lens = np.arange(m) % 5
    lens[-3:] = 60
    A = CsrMatrix.from_host(_ragged(rng, m, lens, 64, np.float64))
    ref = spgemm(A, B).to_host()
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    for r in range(5):
        print("case: %d rows, pass %d" % (m, r), flush=True)
        with torch.cuda.stream(s1):
            plan = Plan(A, B)
        with torch.cuda.stream(s2):
            C = plan.compute()
            s2.synchronize()
        for got, want in zip(C.to_host()[2:], ref[2:]):
            assert np.array_equal(got, want)
        torch.cuda.synchronize()


@pytest.mark.parametrize("sizes", [[1, 2, 5] * 60, [1] * 300 + [900], [700, 256, 257, 1, 300]])
def test_one_shot_batch_copy_parts(sizes):
    """Row tiles full and nearly empty, taken by one work-group and by many,
    with long products per row (two rows per wavefront)."""
    from paper_1504_05022_amd import CsrMatrix, batch_multiply
    rng = np.random.default_rng(len(sizes))
    k = 40
    B = _ragged(rng, k, [20] * k, 500, np.float64)
    As = [_ragged(rng, n, rng.integers(5, 30, n), k, np.float64) for n in sizes]
    print("case: %d problems" % len(sizes), flush=True)
    dB = CsrMatrix.from_host(B)
    out = batch_multiply([(CsrMatrix.from_host(a), dB) for a in As])
    for C, a in zip(out, As):
        _, _, rp, ci, v = C.to_host()
        ref = oracle.spgemm(a.as_tuple(), B.as_tuple())
        assert np.array_equal(rp, ref.row_ptr) and np.array_equal(ci, ref.col_idx)
        assert np.array_equal(v, ref.val)  # Gustavson's order


@pytest.mark.parametrize("streams", ["two", "from default", "to default"])
def test_plan_released_on_another_stream(streams):
    """A plan computed on another stream than it was analysed on and released
    at once: its memory is not handed out before that stream's copy into C,
    which still reads it, has ended."""
    import torch
    from paper_1504_05022_amd import CsrMatrix, Plan, spgemm
    A, _ = S.config2(n=30000, cap=1500)
    M = CsrMatrix.from_host(A)
    ref = spgemm(M, M).to_host()
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    if streams == "from default":
        s1 = torch.cuda.default_stream()
    if streams == "to default":
        s2 = torch.cuda.default_stream()
    for r in range(5):
        print("case: %s, pass %d" % (streams, r), flush=True)
        with torch.cuda.stream(s1):
            plan = Plan(M, M)
            size = plan.info.bytes_scratch
        with torch.cuda.stream(s2):
            C = plan.compute()
            plan.close()
        with torch.cuda.stream(s1):
            for _ in range(4):
                torch.zeros(size, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        for got, want in zip(C.to_host()[2:], ref[2:]):
            assert np.array_equal(got, want)
