"""Kernel branches at the sizes where they can go wrong: tile edges,
remainders, the smallest and largest of each range, against the fp64 oracle
within |err| <= 1e-5 (1 + |A||B|)."""
import numpy as np
import pytest

import gen
import oracle
from spmm_check import assert_close, run

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2608_05033_amd as sd  # noqa: E402


@pytest.mark.parametrize("n", [1, 2, 5, 8, 16, 32, 33, 64, 100, 256, 300])
@pytest.mark.parametrize("steps", [1, 7, 8, 9, 64, 65])
def test_merge_runs(n, steps):
    """Merge-path pieces of `steps` path steps: rows that end on piece and tile
    edges, runs of empty rows longer than a tile of row ends, and rows whose
    carries span 1 to 70 pieces (the fix-up's lane-group and wave paths)."""
    lens = []
    for carries in (1, 2, 3, 4, 5, 6, 8, 9, 16, 17, 33, 70):
        lens += [min(carries * steps, 2000), 0, 1, steps, 0, 0, max(0, steps - 1), 2]
    lens = np.array(lens + [0] * 150 + [1] * 70 + [0, 3, 0], np.int32)
    A = gen.random_rows(lens.size, 2100, lens, seed=steps)
    units = max(1, (A.m + A.nnz) // steps)
    B = gen.dense_uniform(A.k, n, seed=n)
    C64, S = oracle.spmm(A, B)
    print(f"case merge runs n={n} steps={steps} units={units}", flush=True)
    with sd.sd_plan_ex(A, n, force="csr_merge", units=units) as plan:
        for mis in (False, True):
            assert_close(run(sd, plan, B, A.m, misalign=mis), C64, S, f"merge n={n} steps={steps} mis={mis}")


def _device_csr(A):
    return [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (A.rowptr, A.colidx, A.values)]


def _lens(kind):
    rng = np.random.default_rng(7)
    if kind == "strip edges":  # 16-row strips of 511 .. 4097 entries, 8- and 4-row ones on both sides too
        rows = []
        for total in (511, 512, 513, 1024, 1025, 2048, 2049, 4095, 4096, 4097, 9000):
            cut = np.sort(rng.integers(0, total + 1, 15))
            rows += list(np.diff(np.concatenate([[0], cut, [total]])))
        return np.array(rows + [5, 0, 3], np.int32), 5000
    if kind == "windows":  # long strips over several column windows, one of them nearly empty
        return np.array([6000] * 16 + [1] * 13 + [300] * 20 + [20000] + [0] * 7, np.int32), 3 * 131072 + 5
    if kind == "long rows":  # quartiles past the counted lengths
        return np.array([4093, 4094, 4095, 4096, 5000, 7000, 7000, 6999], np.int32), 7000
    if kind == "some long":  # one quartile past them, the others not
        return np.array([3] * 9 + [4095] * 4, np.int32), 4100
    return np.array([512] * 32 + [0] * 40 + [511, 1], np.int32), 512  # "full": dense 16x16 tiles


@pytest.mark.parametrize("kind", ["strip edges", "windows", "long rows", "some long", "full"])
def test_analyze_strips(kind):
    """The device analysis equals the host's byte for byte where strips change
    hands between a wave, a workgroup and column windows, and where the row
    lengths pass the counted range."""
    lens, k = _lens(kind)
    A = gen.random_rows(lens.size, k, lens, seed=3)
    print(f"case analyze {kind} m={A.m} nnz={A.nnz}", flush=True)
    host = sd.sd_analyze(A, raw=True)
    dev = sd.sd_analyze_device(*_device_csr(A), A.m, A.k, A.nnz, raw=True)
    assert bytes(host) == bytes(dev)


@pytest.mark.parametrize("kind", ["strip edges", "windows", "full"])
@pytest.mark.parametrize("what", ["range", "order", "repeat", "negative"])
def test_analyze_strips_bad_columns(kind, what):
    """A column rule broken in a short, a middling or a long strip is found."""
    lens, k = _lens(kind)
    A = gen.random_rows(lens.size, k, lens, seed=3)
    rows = [r for r in range(A.m) if A.rowptr[r + 1] - A.rowptr[r] >= 2]
    for r in (rows[0], rows[len(rows) // 2], rows[-1]):
        col = A.colidx.copy()
        p = A.rowptr[r + 1] - 1
        if what == "range":
            col[p] = A.k
        elif what == "negative":
            col[A.rowptr[r]] = -1
        elif what == "order":
            col[p], col[p - 1] = col[p - 1], col[p]
        else:
            col[p] = col[p - 1]
        bad = gen.CSR(A.m, A.k, A.rowptr, col, A.values)
        with pytest.raises(sd.SparseDittoError) as e:
            sd.sd_analyze_device(*_device_csr(bad), A.m, A.k, A.nnz)
        assert e.value.status == sd.SD_ERR_INVALID_CSR
        with pytest.raises(sd.SparseDittoError) as e:
            sd.sd_plan_device(*_device_csr(bad), A.m, A.k, A.nnz, 8)
        assert e.value.status == sd.SD_ERR_INVALID_CSR


def test_memory_reuse_in_flight():
    """Plans destroyed with their products still in flight, on two streams, and
    rebuilt in the memory they leave: every product is its own plan's."""
    mats = [gen.rmat(12, 60000, seed=s) for s in range(4)]
    dev = [_device_csr(A) for A in mats]
    n = 64
    B = torch.randn(mats[0].k, n, device="cuda")
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    want = []
    for A, d in zip(mats, dev):
        with sd.sd_plan_device(*d, A.m, A.k, A.nnz, n) as plan:
            C = torch.empty(A.m, n, device="cuda")
            sd.sd_spmm(plan, B, C)
            torch.cuda.synchronize()
            want.append(C)
    for turn in range(6):
        got = []
        for i, (A, d) in enumerate(zip(mats, dev)):
            s = streams[(i + turn) % 2]
            plan = sd.sd_plan_device(*d, A.m, A.k, A.nnz, n, stream=s)
            C = torch.empty(A.m, n, device="cuda")
            for _ in range(20):
                sd.sd_spmm(plan, B, C, s)
            plan.destroy()  # without waiting
            got.append(C)
        torch.cuda.synchronize()
        for c, w in zip(got, want):
            assert torch.equal(c, w)
        if turn == 2:
            sd.sd_release_memory()


@pytest.mark.parametrize("fam", ["bsr", "bell"])
@pytest.mark.parametrize("mb", [3, 767, 768, 1100, 2050])
@pytest.mark.parametrize("n", [4, 20, 36, 64, 68, 100, 128, 132, 200, 260])
def test_mfma_column_tiles(fam, mb, n):
    """Every column-tile shape of the MFMA block kernel with a whole and a partial
    last tile: 16, 32 and 64 columns, and 128 from 2,048 waves on, workgroups
    whose waves share a block-row and ones that end inside it."""
    A = gen.block(mb, 40, 16, 2, 30, 0.9, mb)
    A = gen.CSR(A.m - 5, A.k, A.rowptr[:A.m - 4], A.colidx[:A.rowptr[A.m - 5]], A.values[:A.rowptr[A.m - 5]])
    B = gen.dense_uniform(A.k, n, seed=n)
    C64, S = oracle.spmm(A, B)
    print(f"case mfma tiles {fam} mb={mb} n={n}", flush=True)
    with sd.sd_plan_ex(A, n, force=fam, engine="mfma") as plan:
        assert_close(run(sd, plan, B, A.m), C64, S, f"tiles/{fam}/{mb}/{n}")


@pytest.mark.parametrize("shape,n", [("band", n) for n in (33, 64, 96, 130, 256, 300)] +
                         [(shape, n) for shape in ("short", "empty") for n in (80, 96, 125, 256)])
def test_streamed_rows(shape, n):
    """Rows taken by lane groups as they become free: a narrow band (rows of
    several tiles, empty rows, a last workgroup that is not full), short rows on
    any columns, and mostly empty rows; B and C on a 16-byte boundary and off it."""
    rng = np.random.default_rng(n)
    m = k = 66003
    if shape == "band":
        lens = rng.integers(0, 30, m)
        lens[::501] = 150
        lens[1000:1400] = 0
        lens[-1] = 70
        base = np.clip(np.arange(m) - 200, 0, m - 400)
        width = 400
    else:
        m, k = 132003, 30000  # workgroups enough, an upper quartile above 4 entries
        lens = rng.integers(2, 9, m) if shape == "short" else rng.integers(5, 9, m)
        if shape == "empty":
            lens[rng.random(m) < 0.5] = 0
            lens[20000:40000] = 0
        lens[::7001] = 90
        base, width = np.zeros(m, np.int64), k
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows = np.repeat(np.arange(m), lens)
    j = np.arange(rowptr[-1]) - rowptr[rows]
    L = lens[rows]
    lo, hi = j * width // L, (j + 1) * width // L
    col = (base[rows] + lo + rng.integers(0, 1 << 30, rows.size) % np.maximum(1, hi - lo)).astype(np.int32)
    A = gen.CSR(m, k, rowptr, col, rng.uniform(-1, 1, col.size).astype(np.float32))
    B = gen.dense_uniform(k, n, seed=n)
    C64, S = oracle.spmm(A, B)
    print(f"case streamed rows {shape} n={n}", flush=True)
    with sd.sd_plan_ex(A, n, force="csr_row") as plan, sd.sd_plan_ex(A, n, force="csr_row", wg_order=2) as other:
        assert plan.info["stream_rows"] > 0 and other.info["stream_rows"] == 0
        out = run(sd, plan, B, m)
        assert_close(out, C64, S, f"streamed {shape} n={n}")
        # a row is summed in the same order either way
        assert np.array_equal(out.view(np.uint32), run(sd, other, B, m).view(np.uint32))
        assert_close(run(sd, plan, B, m, misalign=True), C64, S, f"streamed misaligned {shape} n={n}")


@pytest.mark.parametrize("n", [132, 190])
def test_streamed_light_rows(n):
    """The split's light rows streamed by whole waves: 16,000 workgroups and a few, the
    last one not full, beside chunks of heavy rows."""
    m, k = 16 * 16003 + 5, 4000
    lens = np.random.default_rng(n).integers(0, 8, m)
    lens[::9001] = 1500
    A = gen.random_rows(m, k, lens.astype(np.int32), seed=n)
    B = gen.dense_uniform(k, n, seed=n)
    C64, S = oracle.spmm(A, B)
    print(f"case streamed light rows n={n}", flush=True)
    kw = dict(force="csr_split", heavy_threshold=500, chunk_nnz=256, col_tile=256)
    with sd.sd_plan_ex(A, n, **kw) as plan, sd.sd_plan_ex(A, n, rows_per_group=1, **kw) as other:
        assert plan.info["stream_rows"] == 4 and other.info["stream_rows"] == 0
        assert plan.info["n_light"] % 16 != 0 and plan.info["n_heavy"] > 20
        out = run(sd, plan, B, m)
        assert_close(out, C64, S, f"streamed light rows n={n}")
        assert np.array_equal(out.view(np.uint32), run(sd, other, B, m).view(np.uint32))


ODD_FAMILIES = [("csr_row", {}), ("csr_row", {"row_slices": 1}), ("csr_split", {"heavy_threshold": 40, "chunk_nnz": 17}),
                ("csr_merge", {"units": 301}), ("bsr", {"engine": "mfma"}), ("bell", {"engine": "valu"}), ("ell", {}),
                ("ell", {"rows_per_group": 4}), ("win", {"heavy_threshold": 200}), ("sell", {})]


def _odd_product(A, fam, opts, n, off, lanes=None):
    """One product with B and C `off` floats past a 16-byte boundary: right, and
    nothing written outside C."""
    B = gen.dense_uniform(A.k, n, seed=n)
    C64, S = oracle.spmm(A, B)
    Bs = torch.empty(A.k * n + off, device="cuda")
    Bs[off:] = torch.from_numpy(B.reshape(-1))
    Cs = torch.full((A.m * n + 16,), -7.0, device="cuda")
    first = 8 + off
    Cd = Cs[first:first + A.m * n].view(A.m, n)
    with sd.sd_plan_ex(A, n, force=fam, **opts) as plan:
        if lanes:
            assert plan.info["lanes_per_row"] // max(1, plan.info["row_slices"]) == lanes
        sd.sd_spmm(plan, Bs[off:], Cd, torch.cuda.current_stream())
        torch.cuda.synchronize()
    assert_close(Cd.cpu().numpy(), C64, S, f"odd {fam} n={n} off={off}")
    assert bool((Cs[:first] == -7.0).all()) and bool((Cs[first + A.m * n:] == -7.0).all())


@pytest.mark.parametrize("fam,opts", ODD_FAMILIES, ids=[f"{f}-{i}" for i, (f, _) in enumerate(ODD_FAMILIES)])
@pytest.mark.parametrize("n", [4, 5, 6, 7, 9, 15, 17, 31, 33, 50, 63, 65, 101, 130, 255, 257])
@pytest.mark.parametrize("off", [0, 1, 2, 3])
def test_odd_widths(fam, opts, n, off):
    """Widths that leave the last lane fewer columns, in one column per lane or four as
    the plan picks for a small matrix, with B and C at every 4-byte offset, rows of up
    to three column passes, and nothing written outside C."""
    rng = np.random.default_rng(5)
    lens = rng.integers(0, 40, 301)
    lens[::50] = 250
    A = gen.random_rows(301, 260, np.minimum(lens, 260).astype(np.int32), seed=1)
    print(f"case odd {fam} {opts} n={n} off={off}", flush=True)
    _odd_product(A, fam, opts, n, off)


@pytest.mark.parametrize("fam,mean", [("csr_row", 7), ("csr_split", 7), ("ell", 4), ("sell", 4), ("csr_merge", 36)])
@pytest.mark.parametrize("n", [5, 7, 9, 15, 17, 18, 19, 31, 33, 63, 65, 101, 127, 130, 255])
def test_odd_widths_four_columns(fam, mean, n):
    """Four columns per lane at widths of no whole 4, with rows enough for the plan to
    pick them."""
    m = 24011
    lens = np.random.default_rng(n).integers(0, 2 * mean + 1, m)
    if fam == "csr_split":
        lens[::4000] = 700
    A = gen.random_rows(m, 900, lens.astype(np.int32), seed=n)
    four = 1
    while four < min(64, -(-n // 4)):
        four *= 2
    if fam == "csr_merge" and n < 16:
        four *= 4  # one column per lane there
    print(f"case odd four {fam} n={n}", flush=True)
    _odd_product(A, fam, {}, n, n % 4, lanes=four)


@pytest.mark.parametrize("fam", ["bsr", "bell"])
@pytest.mark.parametrize("k", [17, 16 * 32, 16 * 33 + 1, 16 * 65536, 16 * 65536 + 1, 2500003])
def test_block_conversion_windows(fam, k):
    """Device block conversion equals the host's where a block-row's columns end on
    a word, a window, or reach over several windows; empty block-rows and rows."""
    lens = np.array([0] * 16 + [min(k, 40)] * 20 + [0, 1, min(k, 300)] + [0] * 20 + [min(k, 7)] * 3, np.int32)
    A = gen.random_rows(lens.size, k, lens, seed=k % 1000)
    A.colidx[A.rowptr[17:37] - 1] = k - 1  # the last column in every row of two block-rows
    print(f"case block conversion {fam} k={k}", flush=True)
    with sd.sd_plan_ex(A, 8, force=fam) as host, \
            sd.sd_plan_device(*_device_csr(A), A.m, A.k, A.nnz, 8, force=fam) as dev:
        assert dev.info["device_built"] == 1
        for what in (sd.SD_EXPORT_BLOCK_COL, sd.SD_EXPORT_BLOCK_VAL) + ((sd.SD_EXPORT_BLOCK_PTR,) if fam == "bsr" else ()):
            assert sd.sd_plan_export(host, what).tobytes() == sd.sd_plan_export(dev, what).tobytes(), what
        B = gen.dense_uniform(k, 8, seed=1)
        assert run(sd, host, B, A.m).tobytes() == run(sd, dev, B, A.m).tobytes()  # the zero block as well


@pytest.mark.parametrize("m, k", [(2, 1), (4095, 5), (4096, 1023), (4097, 1024), (12293, 1 << 20), (70001, 1 << 28),
                                  (1 << 20, 3000), ((1 << 20) + 1, 3000)])
def test_split_order_sort(m, k):
    """The device's orders of light rows and chunks equal the host's: tiles full and
    not, one to three digit passes, many equal columns, the longest list sorted here
    and one more."""
    lens = np.full(m, 1, np.int32)
    lens[::7] = 0
    if k > 40:
        lens[::max(1, m // 5000)] = 33  # heavy from 8: five chunks of at most 8
    A = gen.random_rows(m, k, lens, seed=m % 1000)
    if k >= 1 << 20:  # columns that repeat, over the whole range
        one = lens[np.repeat(np.arange(m), lens)] == 1
        A.colidx[one] = (A.colidx[one] // (k // 97)) * (k // 97) + 5
    print(f"case split order sort m={m} k={k}", flush=True)
    opts = dict(force="csr_split", heavy_threshold=8, chunk_nnz=8, light_order="last_col", chunk_order="mid_col")
    with sd.sd_plan_ex(A, 8, **opts) as host, \
            sd.sd_plan_device(*_device_csr(A), A.m, A.k, A.nnz, 8, **opts) as dev:
        assert dev.info["device_built"] == 1
        for what in range(1, 21):
            try:
                a = sd.sd_plan_export(host, what)
            except sd.SparseDittoError:
                continue
            assert a.tobytes() == sd.sd_plan_export(dev, what).tobytes(), what


def test_analysis_of_the_most_entries():
    """2^31 - 1 entries: a short strip that ends at the last of them is checked and
    counted like any other, and a column out of range in it is found."""
    k, full = 65536, 32768
    lens = torch.full((full + 16,), k, dtype=torch.int64)
    lens[full - 1] = k - 201
    lens[full:full + 8], lens[full + 8:] = 13, 12
    rowptr = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(lens, 0)])
    nnz = int(rowptr[-1])
    assert nnz == 2 ** 31 - 1
    cols = torch.arange(nnz, dtype=torch.int32, device="cuda").remainder_(k)
    cols[nnz - 200:] = torch.cat([torch.arange(int(n)) * 5000 for n in lens[full:]]).int().cuda()
    vals = torch.ones(nnz, device="cuda")
    rp = rowptr.int().cuda()
    print("case analysis of 2^31 - 1 entries", flush=True)
    st = sd.sd_analyze_device(rp, cols, vals, full + 16, k, nnz)
    assert st["nnz"] == nnz and st["row_max"] == k and st["row_min"] == 12 and st["row_q50"] == k
    assert st["nnzb16"] == (full // 16) * (k // 16) + 13
    assert st["nnzb8"] == (full // 8) * (k // 8) + 13 + 12
    assert st["nnzb4"] == (full // 4) * (k // 4) + 2 * 13 + 2 * 12
    assert st["bell16_width"] == k // 16 and st["diag_nnz"] == full and st["col_deg_max"] == full + 16
    cols[nnz - 1] = k
    with pytest.raises(sd.SparseDittoError) as e:
        sd.sd_analyze_device(rp, cols, vals, full + 16, k, nnz)
    assert e.value.status == sd.SD_ERR_INVALID_CSR


@pytest.mark.parametrize("force,opts", [("csr_row", {}), ("csr_split", {}), ("csr_split", {"heavy_threshold": 4000})])
def test_products_of_the_most_entries(force, opts):
    """2^31 - 1 entries: the lanes' steps past the last row's (or chunk's) end pass the
    largest int32.  Every row holds columns 0 .. 2,047, the last one all but column
    2,047, so C's rows are sums of B's (error below 2,048 rounding steps of the sum of
    magnitudes)."""
    k, m = 2048, 2 ** 20
    nnz = m * k - 1
    cols = torch.arange(k, dtype=torch.int32, device="cuda").repeat(m)[:nnz]
    vals = torch.ones(nnz, device="cuda")
    rp = (torch.arange(m + 1, dtype=torch.int64) * k).clamp_(max=nnz).int().cuda()
    for n in (1, 3, 16, 64, 200):
        print(f"case 2^31 - 1 entries {force} {opts} n={n}", flush=True)
        B = torch.rand(k, n, device="cuda")
        C = torch.full((m, n), float("nan"), device="cuda")
        with sd.sd_plan_device(rp, cols, vals, m, k, nnz, n, force=force, **opts) as plan:
            sd.sd_spmm(plan, B, C)
            torch.cuda.synchronize()
        want, last = B.double().sum(0), B[:-1].double().sum(0)
        tol = k * 2.0 ** -24
        assert bool(((C[:-1] - want).abs() <= tol * want).all())
        assert bool(((C[-1] - last).abs() <= tol * last).all())
        del B, C
    sd.sd_release_memory()


def test_merge_path_of_the_most_rows():
    """2^31 - 1 rows, nearly all empty: the last piece's tile of row ends passes the
    largest row number."""
    m, n = 2 ** 31 - 1, 1
    rp = torch.full((m + 1,), 2, dtype=torch.int32, device="cuda")
    rp[0], rp[1:6], rp[m] = 0, 1, 3  # one entry in rows 0, 5 and m - 1
    cols = torch.tensor([1, 0, 2], dtype=torch.int32, device="cuda")
    vals = torch.tensor([2.0, 3.0, 5.0], device="cuda")
    B = torch.tensor([[7.0], [11.0], [13.0]], device="cuda")
    C = torch.full((m, n), -7.0, device="cuda")
    print("case merge path of 2^31 - 1 rows", flush=True)
    sd.sd_spmm_merge_noalloc(rp, cols, vals, m, 3, 3, n, B, C)
    torch.cuda.synchronize()
    assert [float(C[r, 0]) for r in (0, 5, m - 1)] == [22.0, 21.0, 65.0]
    assert int(torch.count_nonzero(C)) == 3


@pytest.mark.parametrize("n", [1, 7, 8, 9, 12, 31])
def test_split_stores_of_small_and_large_outputs(n):
    """Light rows of the narrow split below and above the size of C from which they
    are stored past L2 (2 MiB), whole widths and odd ones."""
    m, k = 60013, 4000
    lens = np.random.default_rng(n).integers(0, 9, m)
    lens[::3001] = 900
    A = gen.random_rows(m, k, lens.astype(np.int32), seed=n)
    B = gen.dense_uniform(k, n, seed=n)
    C64, S = oracle.spmm(A, B)
    print(f"case split stores n={n}", flush=True)
    with sd.sd_plan_ex(A, n, force="csr_split") as plan:
        assert plan.info["n_light"] > 59000 and plan.info["n_heavy"] > 10
        assert_close(run(sd, plan, B, m), C64, S, f"split stores n={n}")


@pytest.mark.parametrize("n", [63, 129, 180, 256, 300])
@pytest.mark.parametrize("rows", [(40, 31), (40, 33), (2000, 500), (4000, 300), (9000, 350)])
def test_merge_long_rows(n, rows):
    """The merge path's batches without a row's end: means just under and over 32,
    rows that end on batch edges, empty rows between long ones, and (the last) enough
    gathered bytes for two workgroups per CU."""
    m, mean = rows
    lens = np.full(m, mean)
    lens[1::7], lens[2::7] = 8 * (mean // 8), 0
    lens[3::7] += mean
    lens[0], lens[-1] = 64, 1
    A = gen.random_rows(m, 1500, lens.astype(np.int32), seed=n)
    B = gen.dense_uniform(A.k, n, seed=n)
    C64, S = oracle.spmm(A, B)
    csr = _device_csr(A)
    Bd, Cd = torch.from_numpy(B).cuda(), torch.full((m, n), float("nan"), device="cuda")
    for units in (0, 1, 37, 999):
        print(f"case merge long rows n={n} rows={rows} units={units}", flush=True)
        Cd.fill_(float("nan"))
        sd.sd_spmm_merge_noalloc(*csr, m, A.k, A.nnz, n, Bd, Cd, units=units)
        torch.cuda.synchronize()
        assert_close(Cd.cpu().numpy(), C64, S, f"merge long n={n} {rows} units={units}")
    with sd.sd_plan_ex(A, n, force="csr_merge") as plan:
        if n > 128:
            assert (plan.info["lds_bytes"] == 65536) == (4.0 * A.nnz * n >= 0.9e9 and A.nnz >= 32 * m)
        elif m == 9000:
            assert plan.info["lds_bytes"] == 65536
        assert_close(run(sd, plan, B, m), C64, S, f"merge long plan n={n} {rows}")
