"""The workgroup kernels of the CSR product with 4, 8 and 16 waves to a row: the sizes on either side of the
lines of the rule (mean row of the right operand, LDS of a row's accumulators), the most LDS a row may take, a
row beyond it, and an arena that only the smallest table of boundaries fits; products with a diagonal; the
matrix-vector product with the vector in LDS; matrices with as many entries as there may be.

A value is a sum of at most as many products as the left operand has entries in a row.  Against the oracle's
product of the same fp32 factors in 64 bits each of them and each addition errs by at most 2^-24 of the sum of the
magnitudes."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import cnn as ocnn

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bp():
    import paper_1907_10134_amd as bp
    return bp


def _rows(rows, cols, per_row, rng):
    """`per_row` distinct columns in every row, except the second, which is empty, and the third, which is full
    up to 2000 columns."""
    idx = []
    for r in range(rows):
        n = 0 if r == 1 else min(cols, 2000) if r == 2 else per_row
        idx.append(np.sort(rng.choice(cols, n, replace=False)))
    indptr = np.cumsum([0] + [len(i) for i in idx])
    data = rng.standard_normal(indptr[-1]).astype(np.float32)
    return sp.csr_matrix((data, np.concatenate(idx), indptr), shape=(rows, cols))


def _to_gpu(bp, m):
    import torch
    return bp.CsrMatrix(m.shape[0], m.shape[1], torch.from_numpy(m.indptr.astype(np.int32)).cuda(),
                        torch.from_numpy(m.indices.astype(np.int32)).cuda(), torch.from_numpy(m.data.astype(np.float32)).cuda())


# columns of the right operand, entries of most of its rows (the mean is some 10 more), entries a row of the left
# one, which kernel
CASES = [
    (2100, 620, 100, "dense, 4 waves below 640"), (2100, 660, 100, "dense, 16 waves"),
    (5121, 80, 100, "dense, 4 waves below 96"), (5121, 110, 100, "dense, 8 waves above 20 KB"),
    (5120, 110, 100, "dense, 4 waves at 20 KB"), (10241, 180, 100, "dense, 8 waves below 200"),
    (10241, 215, 100, "dense, 16 waves above 40 KB"), (10240, 215, 100, "dense, 8 waves at 40 KB"),
    (40960, 700, 100, "dense, 16 waves and all of the LDS"), (40961, 700, 100, "staged, 16 waves"),
    (100000, 150, 30, "staged, 8 waves"), (100000, 230, 30, "staged, 16 waves above 40 KB"),
    (150000, 1200, 40, "global, 16 waves"),
]


@pytest.mark.parametrize("cols,per_row,left_row,what", CASES, ids=[c[3] for c in CASES])
def test_products_by_rows_of_four_to_sixteen_waves(bp, cols, per_row, left_row, what):
    import torch
    rng = np.random.default_rng(cols + per_row)
    right = _rows(150, cols, per_row, rng)
    left = _rows(67, 150, left_row, rng)
    left = sp.csr_matrix(left.multiply(np.arange(67)[:, None] != 2))          # without the full row
    left.eliminate_zeros()
    left = left.astype(np.float32)
    ref = ocnn.csr_product(left.astype(np.float64), right.astype(np.float64))
    size = ocnn.csr_product(abs(left).astype(np.float64), abs(right).astype(np.float64))
    d0 = sp.csr_matrix(rng.standard_normal((cols, 2)).astype(np.float32))
    d3 = sp.csr_matrix(rng.standard_normal((5, 67)).astype(np.float32))
    d4 = sp.csr_matrix(rng.standard_normal((4, 5)).astype(np.float32))
    jts = [_to_gpu(bp, m) for m in (d0, right, left, d3, d4)]
    seed = torch.from_numpy(rng.standard_normal(2).astype(np.float32)).cuda()
    grads = [torch.empty((m.rows,), dtype=torch.float32, device="cuda") for m in jts]

    def values(plan):
        out = []
        for _ in range(2):
            plan.run(jts, seed, grads)
            torch.cuda.synchronize()
            for k in range(plan.num_products()):
                got, l, r = plan.product(k)
                if (l, r) == (2, 1):
                    np.testing.assert_array_equal(got.indptr.cpu().numpy(), ref.indptr)
                    np.testing.assert_array_equal(got.indices.cpu().numpy(), ref.indices)
                    out.append(got.data.cpu().numpy().copy())
        assert len(out) == 2 and np.array_equal(out[0], out[1])
        return out[0]

    plan = bp.SpscanPlan(jts, 1, torch.empty((1 << 28,), dtype=torch.uint8, device="cuda"))
    bound = (left_row + 2) * 2.0**-24 * size.data          # the second order of the bound: one more
    assert np.all(np.abs(values(plan) - ref.data) <= bound)
    used = plan.arena_used()
    plan.close()
    # an arena of what four ways take: 3 boundaries a row of the right operand, whatever the rule prefers, and no columns
    # in 16 bits
    more = {4: 0, 8: 4, 16: 12}
    copied = (2 * right.nnz + 255) // 256 * 256 if what.startswith("dense") else 0
    for ways in (8, 16):
        if ("%d waves" % ways) in what:
            room = used - copied - 4 * 150 * more[ways] + 255
            plan = bp.SpscanPlan(jts, 1, torch.empty((room,), dtype=torch.uint8, device="cuda"))
            assert plan.arena_used() <= room
            assert np.all(np.abs(values(plan) - ref.data) <= bound)
            plan.close()


@pytest.mark.parametrize("cols,per_row,left_row", [(2100, 200, 63), (2100, 200, 64), (2100, 70, 128), (2101, 70, 129),
                                                   (5121, 110, 192), (10240, 215, 130), (40960, 700, 100)])
def test_dense_products_with_columns_in_16_bits(bp, cols, per_row, left_row):
    """Batches of exactly 64 entries of a row (walked without looking for the next one), one fewer and one more, a row
    whose entries clear and fill a small part of the accumulators, columns that are no multiple of 64; then an arena
    without room for the copy of the columns: the same bits, and both within the bound of the sums."""
    import torch
    rng = np.random.default_rng(cols + left_row)
    right = _rows(200, cols, per_row, rng)
    left = _rows(40, 200, left_row, rng).tolil()
    left[2] = 0
    left[3, :197] = 0                            # few entries
    left = sp.csr_matrix(left).astype(np.float32)
    left.eliminate_zeros()
    ref = ocnn.csr_product(left.astype(np.float64), right.astype(np.float64))
    size = ocnn.csr_product(abs(left).astype(np.float64), abs(right).astype(np.float64))
    d0 = sp.csr_matrix(rng.standard_normal((cols, 2)).astype(np.float32))
    d3 = sp.csr_matrix(rng.standard_normal((5, 40)).astype(np.float32))
    d4 = sp.csr_matrix(rng.standard_normal((4, 5)).astype(np.float32))
    jts = [_to_gpu(bp, m) for m in (d0, right, left, d3, d4)]
    seed = torch.from_numpy(rng.standard_normal(2).astype(np.float32)).cuda()
    grads = [torch.empty((m.rows,), dtype=torch.float32, device="cuda") for m in jts]
    used, values = 1 << 28, []
    for room in ("all", "without"):
        if room == "without":
            used -= 2 * right.nnz // 256 * 256
        plan = bp.SpscanPlan(jts, 1, torch.empty((used,), dtype=torch.uint8, device="cuda"))
        plan.run(jts, seed, grads)
        torch.cuda.synchronize()
        got = [plan.product(k)[0] for k in range(plan.num_products()) if plan.product(k)[1:] == (2, 1)]
        assert len(got) == 1
        values.append(got[0].data.cpu().numpy().copy())
        assert room == "all" or plan.arena_used() < before
        before = used = plan.arena_used()
        plan.close()
    assert np.all(np.abs(values[0] - ref.data) <= (left_row + 2) * 2.0**-24 * size.data)
    assert np.array_equal(values[0], values[1])


@pytest.mark.parametrize("cols,rows,per_row,ways", [(2100, 2000, 200, 4), (5121, 1500, 110, 8)])
def test_an_arena_smaller_than_the_columns_in_16_bits(bp, cols, rows, per_row, ways):
    """Few rows by a large right operand: the copy of its columns takes more than all else that the plan asks for.  The
    arena that a plan without it, and then with the boundaries of four ways, needs is enough to the byte, and one unit
    of 256 bytes less is not."""
    import torch
    rng = np.random.default_rng(cols)
    right = _rows(rows, cols, per_row, rng)
    left = sp.csr_matrix(rng.standard_normal((3, rows)).astype(np.float32))
    ref = ocnn.csr_product(left.astype(np.float64), right.astype(np.float64))
    size = ocnn.csr_product(abs(left).astype(np.float64), abs(right).astype(np.float64))
    tails = [sp.csr_matrix(rng.standard_normal(shape).astype(np.float32)) for shape in ((5, 3), (4, 5))]
    jts = [_to_gpu(bp, m) for m in (sp.csr_matrix(rng.standard_normal((cols, 2)).astype(np.float32)), right, left, *tails)]
    seed = torch.from_numpy(rng.standard_normal(2).astype(np.float32)).cuda()
    grads = [torch.empty((m.rows,), dtype=torch.float32, device="cuda") for m in jts]

    def unit(n):
        return (n + 255) // 256 * 256

    def values(arena_bytes):
        plan = bp.SpscanPlan(jts, 1, torch.empty((arena_bytes,), dtype=torch.uint8, device="cuda"))
        plan.run(jts, seed, grads)
        torch.cuda.synchronize()
        got = [plan.product(k)[0] for k in range(plan.num_products()) if plan.product(k)[1:] == (2, 1)]
        out, used = got[0].data.cpu().numpy().copy(), plan.arena_used()
        plan.close()
        return out, used

    first, used = values(1 << 28)
    assert np.all(np.abs(first - ref.data) <= (rows + 2) * 2.0**-24 * size.data)
    without = used - unit(2 * right.nnz)
    assert without < unit(2 * right.nnz)
    least = without - unit(4 * (ways - 1) * rows) + unit(4 * 3 * rows)
    for room in {without, least}:
        got, then = values(room)
        assert then == room and np.all(np.abs(got - ref.data) <= (rows + 2) * 2.0**-24 * size.data)
        assert room == least != without or np.array_equal(got, first)      # (fewer ways: another order of the sums)
    with pytest.raises(bp.BppsaError):
        values(least - 256)


def _diagonal(n, rng):
    return sp.csr_matrix((rng.standard_normal(n).astype(np.float32), np.arange(n), np.arange(n + 1)), shape=(n, n))


@pytest.mark.parametrize("side", ["left", "right", "both", "almost", "permutation"])
@pytest.mark.parametrize("per_row,rows", [(1, 1), (3, 65), (64, 33), (65, 5), (300, 401)])
def test_products_with_a_diagonal(bp, side, per_row, rows):
    """A diagonal on either side scales the other factor, whose rows may be empty; a diagonal but for one entry and
    a permutation of as many entries are no diagonals.  Every value is one product: equal to numpy's."""
    import torch
    rng = np.random.default_rng(7 * rows + per_row)
    cols = 500
    other = _rows(rows, cols, per_row, rng) if rows > 2 else sp.csr_matrix(np.eye(1, cols, 3, dtype=np.float32) * 2)
    n = rows if side == "left" else cols
    d = _diagonal(n, rng)
    if side == "almost" and n > 1:
        d.indices[-1] = 0                        # the last row reads the first column
    elif side == "permutation":
        d.indices[:] = d.indices[::-1]
    if side == "left":
        left, right = d, other
    elif side == "both":
        left, right = d, _diagonal(n, rng)
    else:
        left, right = other, d
    ref = ocnn.csr_product(left, right)
    d0 = sp.csr_matrix(rng.standard_normal((right.shape[1], 2)).astype(np.float32))
    d3 = sp.csr_matrix(rng.standard_normal((5, left.shape[0])).astype(np.float32))
    d4 = sp.csr_matrix(rng.standard_normal((4, 5)).astype(np.float32))
    jts = [_to_gpu(bp, m) for m in (d0, right, left, d3, d4)]
    plan = bp.SpscanPlan(jts, 1, torch.empty((1 << 26,), dtype=torch.uint8, device="cuda"))
    grads = [torch.empty((m.rows,), dtype=torch.float32, device="cuda") for m in jts]
    seen = 0
    for again in range(2):                       # the second time with other values on the same plan
        if again:
            jts[1].data.mul_(3.0)
            jts[2].data.neg_()
        plan.run(jts, torch.ones(2, device="cuda"), grads)
        torch.cuda.synchronize()
        for k in range(plan.num_products()):
            got, l, r = plan.product(k)
            if (l, r) != (2, 1):
                continue
            seen += 1
            np.testing.assert_array_equal(got.indptr.cpu().numpy(), ref.indptr)
            np.testing.assert_array_equal(got.indices.cpu().numpy(), ref.indices)
            a = sp.csr_matrix((jts[2].data.cpu().numpy(), left.indices, left.indptr), shape=left.shape)
            b = sp.csr_matrix((jts[1].data.cpu().numpy(), right.indices, right.indptr), shape=right.shape)
            want = ocnn.csr_product(a, b).data
            if side in ("left", "right", "both"):
                np.testing.assert_array_equal(got.data.cpu().numpy(), want)
            else:                                # two entries of a row may meet in the first column
                np.testing.assert_allclose(got.data.cpu().numpy(), want, rtol=0, atol=3 * 2.0**-24 * 50)
    assert seen == 2
    plan.close()


@pytest.mark.parametrize("rows,cols,per_row", [
    (8193, 4096, 300), (12600, 4097, 192), (12600, 4095, 192), (8192, 8192, 293), (4096, 8193, 600), (4111, 20480, 620),
    (9000, 20481, 270), (4096, 40960, 590), (4100, 40961, 590), (20011, 12000, 193)])
def test_spmv_with_the_vector_in_lds(bp, rows, cols, per_row):
    """Either side of the rule for keeping the vector in LDS; rows of every length from none to three times the
    mean.  A row of n products, fp32, in n additions at most: n + 1 roundings of the sum of the magnitudes."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(rows + cols)
    lengths = torch.full((rows,), per_row, device="cuda")
    lengths[1], lengths[2], lengths[3], lengths[rows - 1] = 0, min(3 * per_row, cols), 1, 64
    lengths[4:40] = torch.arange(239, 275, device="cuda")             # around the four entries of 64 lanes
    indptr = torch.zeros(rows + 1, dtype=torch.int64, device="cuda")
    indptr[1:] = lengths.cumsum(0)
    nnz = int(indptr[-1])
    row = torch.repeat_interleave(torch.arange(rows, device="cuda"), lengths)
    place = torch.arange(nnz, device="cuda") - indptr[row]
    indices = place * (cols // lengths.clamp(min=1))[row]             # ascending; the last column in some row
    indices[indptr[3]] = cols - 1
    data = torch.randn(nnz, device="cuda", generator=g)
    x = torch.randn(cols, device="cuda", generator=g)
    A = bp.CsrMatrix(rows, cols, indptr.int(), indices.int(), data)
    y = torch.full((rows,), 7.0, device="cuda")
    bp.spmv(A, x, y)
    t = data.double() * x.double()[indices]
    ref = torch.zeros(rows, dtype=torch.float64, device="cuda").index_add_(0, row, t)
    size = torch.zeros(rows, dtype=torch.float64, device="cuda").index_add_(0, row, t.abs())
    assert bool(((y.double() - ref).abs() <= (lengths + 2) * 2.0**-24 * size).all())
    assert float(y[1]) == 0.0


# ---- 2^31 - 2 entries, the most that is accepted: positions past the end of the last row are beyond 31 bits --------
MOST = 2**31 - 2


def _full_rows(bp, rows, length, cols, free=0):
    """Rows of `length` entries in the columns 0 .. length - 1, all 1, the first two entries shorter; `free` bytes of
    memory are wanted besides."""
    import torch
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < (18 << 30) + 12 * rows + free:
        pytest.skip("not enough memory")
    assert rows * length == MOST + 2
    indices = torch.empty(MOST, dtype=torch.int32, device="cuda")
    at = torch.arange(length, dtype=torch.int32, device="cuda")
    indices[:length - 2] = at[:length - 2]
    indices[length - 2:].view(rows - 1, length)[:] = at
    indptr = torch.arange(-2, MOST + 1, length, dtype=torch.int64, device="cuda").clamp_(min=0).int()
    assert indptr.numel() == rows + 1
    return bp.CsrMatrix(rows, cols, indptr, indices, torch.ones(MOST, dtype=torch.float32, device="cuda"))


@pytest.mark.parametrize("length,cols", [(32768, 40960), (32768, 50000), (128, 128), (32, 32), (8, 8), (2, 2)])
def test_spmv_of_as_many_entries_as_there_may_be(bp, length, cols):
    """Every form of the kernel by the mean of the rows.  Whole numbers below 2^24: exact."""
    import torch
    A = _full_rows(bp, 2**31 // length, length, cols)
    x = (torch.arange(cols, device="cuda") % 5).float()
    y = torch.full((A.rows,), 7.0, device="cuda")
    bp.spmv(A, x, y)
    assert float(y[0]) == float(x[:length - 2].sum())
    assert bool((y[1:] == x[:length].sum()).all())


@pytest.mark.parametrize("side", ["left, one entry a row", "left, block", "right, scaled", "right, single", "right, block"])
def test_products_with_as_many_entries_as_there_may_be(bp, side):
    """Either factor of a product, in the kernels that walk its rows.  Whole numbers below 2^24: exact."""
    import torch
    length, rows = 4096, 2**19
    big = _full_rows(bp, rows, length, length, 40 << 30)
    dev = dict(device="cuda")

    def csr(rows, cols, per_row, columns):
        n = rows * per_row
        return bp.CsrMatrix(rows, cols, torch.arange(0, n + 1, per_row, dtype=torch.int32, **dev),
                            columns.to(torch.int32), (1 + torch.arange(n, **dev) % 3).float())
    if side.startswith("left"):
        width = 1 if "one" in side else 1100         # rows of the product: one entry, and more than a wave takes
        left, right = big, csr(length, width, 1, torch.arange(length, **dev) % width)
    else:
        n, per_row, columns = {"right, scaled": (rows, 1, torch.arange(rows, **dev)),
                               "right, single": (rows, 1, torch.arange(rows, **dev).flip(0)),
                               "right, block": (2, 2, torch.arange(rows - 4, rows, **dev))}[side]
        left, right = csr(n, rows, per_row, columns), big
    d0 = csr(right.cols, 1, 1, torch.zeros(right.cols, **dev))
    d3 = csr(1, left.rows, 1, torch.zeros(1, **dev))
    d4 = csr(1, 1, 1, torch.zeros(1, **dev))
    jts = [d0, right, left, d3, d4]
    arena = torch.empty((30 << 30,), dtype=torch.uint8, **dev)
    plan = bp.SpscanPlan(jts, 1, arena)
    plan.run(jts, torch.ones(1, **dev), [torch.empty(m.rows, **dev) for m in jts])
    torch.cuda.synchronize()
    got = [plan.product(k)[0] for k in range(plan.num_products()) if plan.product(k)[1:] == (2, 1)]
    assert len(got) == 1
    c = got[0]
    if side.startswith("left"):
        want = torch.zeros(width, **dev).index_add_(0, right.indices.long(), right.data)
        first = torch.zeros(width, **dev).index_add_(0, right.indices.long()[:-2], right.data[:-2])
        assert bool((c.data[:width] == first).all()) and bool((c.data[width:].view(-1, width) == want).all())
    elif "block" in side:
        f = left.data.view(2, 2).sum(1, keepdim=True)
        assert bool((c.data.view(2, length) == f).all())
    else:
        ends = c.indptr.long()
        lengths = ends[1:] - ends[:-1]
        assert bool((c.data == torch.repeat_interleave(left.data, lengths)).all())
    plan.close()
