"""GPU parity: every plan family through the C ABI against the fp64 oracle,
element by element, within |err| <= 1e-5 (1 + |A||B|), at sizes that span
several workgroups and a ragged tail, plus edge cases and determinism."""
import numpy as np
import pytest

import gen
import oracle
from spmm_check import assert_close, expected_csr_arrays, run

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU container
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2608_05033_amd as sd  # noqa: E402


def ragged(m, k, seed, giant=True):
    rng = np.random.default_rng(seed)
    r = rng.integers(0, 60, m)
    r[rng.random(m) < 0.15] = 0
    if giant and m > 10:
        r[m // 2] = min(k, 3000)
        r[m - 1] = min(k, 700)
    return np.minimum(r, k)


MATRICES = {
    "ragged": lambda: gen.random_rows(2000, 3001, ragged(2000, 3001, 1), seed=1),
    "uniform": lambda: gen.uniform_rows(1024, 1024, 8, 0),
    "rmat": lambda: gen.rmat(13, 120000, seed=3),
    "laplace": lambda: gen.laplacian3d(12, 10, 9),
    "block": lambda: gen.block(70, 75, 16, 12, 20, 0.9, 5),
}
_cache = {}


def matrix(name):
    if name not in _cache:
        _cache[name] = MATRICES[name]()
    return _cache[name]


FAMILY_OPTS = [
    ("csr_row", {}),
    ("csr_split", {"heavy_threshold": 40, "chunk_nnz": 17}),
    ("csr_split", {"heavy_threshold": 1, "chunk_nnz": 256}),
    ("csr_split", {"heavy_threshold": 40, "chunk_nnz": 17, "chunk_order": "list"}),
    ("csr_merge", {"units": 97}),
    ("csr_merge", {"units": 5000}),
    ("bsr", {"engine": "valu"}),
    ("bell", {"engine": "valu"}),
    ("ell", {}),
    ("ell", {"rows_per_group": 4}),
    ("ell", {"rows_per_group": 16}),
    ("win", {}),
    ("win", {"heavy_threshold": 40, "chunk_nnz": 17, "window_rows": 16}),
    ("sell", {}),
    ("sell", {"sell_sigma": 1}),
]


@pytest.mark.parametrize("mname", list(MATRICES))
@pytest.mark.parametrize("fam,opts", FAMILY_OPTS, ids=[f"{f}-{i}" for i, (f, _) in enumerate(FAMILY_OPTS)])
@pytest.mark.parametrize("n", [1, 3, 8, 32, 64, 128])
def test_family_parity(mname, fam, opts, n):
    A = matrix(mname)
    if fam in ("bsr", "bell") and mname in ("rmat",) and n > 32:
        pytest.skip("block formats on a power-law graph: large fill, covered at small n")
    B = gen.dense_normal(A.k, n, seed=n)
    print(f"case {mname} {fam} {opts} n={n}", flush=True)
    with sd.sd_plan_ex(A, n, force=fam, **opts) as plan:
        C = run(sd, plan, B, A.m)
    C64, S = oracle.spmm(A, B)
    assert_close(C, C64, S, f"{mname}/{fam}/{n}")


@pytest.mark.parametrize("mname", ["block", "ragged", "laplace"])
@pytest.mark.parametrize("fam", ["bsr", "bell"])
@pytest.mark.parametrize("n", [1, 3, 8, 13, 16, 24, 32, 40, 48, 64, 80, 96, 100, 128, 160, 192, 200, 256])
def test_block_mfma_parity(mname, fam, n):
    """MFMA column tiles of 64, 32 and 16 (partial last tile), of single floats below
    4 columns; B and C on a 16-byte boundary and off it."""
    A = matrix(mname)
    B = gen.dense_uniform(A.k, n, seed=7)
    print(f"case mfma {mname} {fam} n={n}", flush=True)
    with sd.sd_plan_ex(A, n, force=fam, engine="mfma") as plan:
        assert plan.info["engine"] == sd.SD_ENGINE_MFMA
        C, C2 = run(sd, plan, B, A.m, repeat=2)
        Cm = run(sd, plan, B, A.m, misalign=True)
    assert C.tobytes() == C2.tobytes(), "block kernel not deterministic"
    C64, S = oracle.spmm(A, B)
    assert_close(C, C64, S, f"mfma/{mname}/{fam}/{n}")
    assert_close(Cm, C64, S, f"mfma misaligned/{mname}/{fam}/{n}")


@pytest.mark.parametrize("fam,engine", [("bsr", "mfma"), ("bell", "mfma"), ("bsr", "valu"), ("bell", "valu")])
@pytest.mark.parametrize("n", [1, 16, 24, 64, 100, 128])
def test_block_nonfinite_unused_b_rows(fam, engine, n):
    """Rows of B that no nonzero uses may hold Inf or NaN: block-column 0 of A
    is empty, B rows 0..15 are non-finite, and every other B row is finite.
    The CSR product is finite everywhere, and so must be every block plan's,
    including the slots that have no B row (rows past K, Blocked-ELL padding,
    rounds past a block-row's end)."""
    base = gen.block(40, 47, 16, 6, 9, 0.8, 11)
    m, k = base.m - 7, base.k - 5  # ragged last block-row and block-column
    rows = []
    rng = np.random.default_rng(4)
    for i in range(m):
        cols = base.colidx[base.rowptr[i]:base.rowptr[i + 1]]
        cols = cols[(cols >= 16) & (cols < k)]
        if i % 16 == 3:  # uneven block counts per block-row
            cols = cols[: rng.integers(0, cols.size + 1)]
        rows.append(cols)
    lens = np.array([c.size for c in rows])
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colidx = np.concatenate(rows).astype(np.int32)
    A = gen.CSR(m, k, rowptr, colidx, rng.uniform(-1, 1, colidx.size).astype(np.float32))
    B = gen.dense_uniform(k, n, seed=2)
    B[0:16:2] = np.inf
    B[1:16:2] = np.nan
    plan = sd.sd_plan_ex(A, n, force=fam, engine=engine)
    print(f"case nonfinite unused B rows {fam}/{engine} n={n}", flush=True)
    C = run(sd, plan, B, m)
    plan.destroy()
    C64, S = oracle.spmm(A, B)
    assert np.isfinite(C64).all()
    assert_close(C, C64, S, f"{fam}/{engine}/n={n}")


@pytest.mark.parametrize("fam", ["csr_row", "csr_split", "csr_merge", "bsr", "ell", "win", "sell"])
@pytest.mark.parametrize("n", [4, 64, 128, 320, 1000])
def test_wide_and_misaligned(fam, n):
    """n above one column tile (320 needs two tiles of 256), and buffers 4 bytes
    off a 16-byte boundary."""
    A = matrix("ragged")
    B = gen.dense_uniform(A.k, n, seed=11)
    C64, S = oracle.spmm(A, B)
    print(f"case wide {fam} n={n}", flush=True)
    with sd.sd_plan_ex(A, n, force=fam, heavy_threshold=50, chunk_nnz=64, units=301) as plan:
        for mis in (False, True):
            C = run(sd, plan, B, A.m, misalign=mis)
            assert_close(C, C64, S, f"{fam}/{n}/misaligned={mis}")


@pytest.mark.parametrize("fam", ["auto", "csr_row", "csr_split", "csr_merge", "bsr", "bell", "ell", "win", "sell"])
def test_edge_matrices(fam):
    n = 16
    cases = [
        gen.random_rows(37, 19, np.zeros(37, np.int32), seed=1),              # nnz = 0: C must be zeroed
        gen.random_rows(1, 5000, np.array([5000], np.int32), seed=2),         # one full row
        gen.random_rows(5, 1, np.array([1, 0, 1, 1, 0], np.int32), seed=3),   # k = 1
        gen.random_rows(300, 40, np.full(300, 40, np.int32), seed=4),         # dense
        gen.random_rows(17, 33, np.arange(17, dtype=np.int32) * 2, seed=5),   # m, k not multiples of 16
    ]
    for idx, A in enumerate(cases):
        B = gen.dense_uniform(A.k, n, seed=idx)
        print(f"case edge {fam} #{idx} m={A.m} k={A.k} nnz={A.nnz}", flush=True)
        with sd.sd_plan_ex(A, n, force=fam, heavy_threshold=8, chunk_nnz=5, units=7) as plan:
            C = run(sd, plan, B, A.m)
        C64, S = oracle.spmm(A, B)
        assert_close(C, C64, S, f"edge {idx} {fam}")


def test_empty_output_dimensions():
    """m = 0 is a no-op; k = 0 (no nonzeros possible) zero-fills C."""
    A0 = gen.CSR(0, 10, np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32))
    with sd.sd_plan(A0, 8) as plan:
        B = torch.zeros((10, 8), device="cuda")
        C = torch.zeros((0, 8), device="cuda")
        sd.sd_spmm(plan, B, C)
    Ak = gen.CSR(6, 0, np.zeros(7, np.int32), np.zeros(0, np.int32), np.zeros(0, np.float32))
    with sd.sd_plan(Ak, 8) as plan:
        C = torch.full((6, 8), float("nan"), device="cuda")
        sd.sd_spmm(plan, None, C)
        torch.cuda.synchronize()
        assert torch.all(C == 0)


def _lanes(n):
    """Lanes per row of whole widths and of n < 4."""
    lanes = -(-n // 4) if n % 4 == 0 else n
    g = 1
    while g < lanes and g < 64:
        g *= 2
    return g


SLICE_OPTS = [("csr_row", {}), ("csr_split", {"heavy_threshold": 40, "chunk_nnz": 17}),
              ("csr_split", {"heavy_threshold": 1, "chunk_nnz": 256})]


@pytest.mark.parametrize("mname", list(MATRICES))
@pytest.mark.parametrize("fam,opts", SLICE_OPTS, ids=[f"{f}-{i}" for i, (f, _) in enumerate(SLICE_OPTS)])
@pytest.mark.parametrize("n", [1, 3, 8, 16, 32])
@pytest.mark.parametrize("S", [2, 4, 8, 16, 32, 64])
def test_row_slices_parity(mname, fam, opts, n, S):
    """Rows shared by S lane groups (narrow widths) against the oracle."""
    G = _lanes(n)
    if G > 8 or G * S > 64:
        pytest.skip("no sliced geometry for this width")
    A = matrix(mname)
    B = gen.dense_uniform(A.k, n, seed=S)
    print(f"case slices {mname} {fam} {opts} n={n} S={S}", flush=True)
    with sd.sd_plan_ex(A, n, force=fam, row_slices=S, **opts) as plan:
        assert plan.info["row_slices"] == S
        C = run(sd, plan, B, A.m)
        Cm = run(sd, plan, B, A.m, misalign=True)
    C64, S_ = oracle.spmm(A, B)
    assert_close(C, C64, S_, f"slices {mname} {fam} n={n} S={S}")
    assert_close(Cm, C64, S_, f"slices misaligned {mname} {fam} n={n} S={S}")


@pytest.mark.parametrize("mname", ["rmat", "ragged"])
@pytest.mark.parametrize("n", [1, 8, 64, 128])
def test_light_order_changes_no_bits(mname, n):
    """The light-row order only changes which rows run together: each row is
    summed in the same order, so C is bitwise the same either way."""
    A = matrix(mname)
    B = gen.dense_normal(A.k, n, seed=41)
    print(f"case light order {mname} n={n}", flush=True)
    out = {}
    for order in ("ascending", "last_col"):
        with sd.sd_plan_ex(A, n, force="csr_split", heavy_threshold=40, chunk_nnz=64, light_order=order) as plan:
            out[order] = run(sd, plan, B, A.m)
    assert np.array_equal(out["ascending"].view(np.uint32), out["last_col"].view(np.uint32))
    C64, S = oracle.spmm(A, B)
    assert_close(out["last_col"], C64, S, f"light order {mname} n={n}")


@pytest.mark.parametrize("mname", ["rmat", "ragged"])
@pytest.mark.parametrize("n", [1, 8, 64, 128])
def test_chunk_order_changes_no_bits(mname, n):
    """The chunk order only changes which chunks run together: each chunk's
    partial lands in its own workspace row and each row adds its partials in
    chunk order, so C is bitwise the same either way."""
    A = matrix(mname)
    B = gen.dense_normal(A.k, n, seed=43)
    print(f"case chunk order {mname} n={n}", flush=True)
    out = {}
    for order in ("list", "mid_col"):
        with sd.sd_plan_ex(A, n, force="csr_split", heavy_threshold=30, chunk_nnz=7, chunk_order=order) as plan:
            assert plan.info["n_chunks"] > 100
            out[order] = run(sd, plan, B, A.m)
    assert np.array_equal(out["list"].view(np.uint32), out["mid_col"].view(np.uint32))
    C64, S = oracle.spmm(A, B)
    assert_close(out["mid_col"], C64, S, f"chunk order {mname} n={n}")


def test_overlapping_operands_rejected():
    """B and C that share bytes are refused before any launch; adjacent ones are fine."""
    A = matrix("ragged")
    n = 8
    with sd.sd_plan(A, n) as plan:
        buf = torch.zeros((A.k + A.m) * n, device="cuda")
        B, C = buf[: A.k * n], buf[A.k * n:]
        for off in (1, A.k * n // 2):  # C starts inside B
            with pytest.raises(sd.SparseDittoError) as e:
                sd.sd_spmm(plan, B.data_ptr(), C.data_ptr() - 4 * off)
            assert e.value.status == sd.SD_ERR_INVALID_VALUE
        with pytest.raises(sd.SparseDittoError):
            sd.sd_spmm(plan, B, B)
        B.copy_(torch.from_numpy(gen.dense_uniform(A.k, n, seed=4).reshape(-1)).cuda())
        sd.sd_spmm(plan, B, C)  # adjacent, not overlapping
        torch.cuda.synchronize()
        C64, S = oracle.spmm(A, B.view(A.k, n).cpu().numpy())
        assert_close(C.view(A.m, n).cpu().numpy(), C64, S, "adjacent B and C")


@pytest.mark.parametrize("fam", ["csr_row", "csr_split", "csr_merge", "bsr", "ell", "win", "sell"])
def test_deterministic(fam):
    """No atomics anywhere: two runs give bitwise-equal C."""
    A = matrix("rmat")
    B = gen.dense_normal(A.k, 64, seed=5)
    with sd.sd_plan_ex(A, 64, force=fam, heavy_threshold=32, chunk_nnz=32, units=999) as plan:
        C1, C2 = run(sd, plan, B, A.m, repeat=2)
    assert np.array_equal(C1.view(np.uint32), C2.view(np.uint32))


@pytest.mark.parametrize("fam", ["csr_row", "csr_split", "csr_merge", "bsr", "ell", "win", "sell"])
def test_transpose_plan(fam):
    A = matrix("ragged")
    n = 64
    Bt = gen.dense_normal(A.m, n, seed=9)
    with sd.sd_plan_ex(A, n, force=fam, transpose=True, heavy_threshold=30, chunk_nnz=30, units=400) as plan:
        C = run(sd, plan, Bt, A.k)
        if fam not in ("bsr", "ell", "win", "sell"):
            tr, tc, tv = oracle.transpose(A)
            tr, tc, tv = expected_csr_arrays(gen.CSR(A.k, A.m, tr, tc, tv), plan.info)
            assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_ROWPTR), tr)
            assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_COLIDX), tc)
            assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_VALUES).view(np.uint32), tv.view(np.uint32))
    C64, S = oracle.spmm_transposed(A, Bt)
    assert_close(C, C64, S, f"transpose/{fam}")


def test_device_exports_match_oracle():
    """The arrays uploaded to the device are the oracle's conversions, bit for bit."""
    A = matrix("rmat")
    with sd.sd_plan_ex(A, 32, force="csr_split", heavy_threshold=100, chunk_nnz=60) as plan:
        light, chunks = oracle.heavy_split(A.rowptr, A.m, 100, 60)
        light = oracle.light_by_last_col(A, light)
        lptr, col, val, chunks = oracle.split_layout(A, 100, 60, light)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_LIGHT_ROWS), light)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_CHUNKS).reshape(-1, 3), chunks)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_ROWPTR), lptr)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_COLIDX), col)
    with sd.sd_plan_ex(A, 32, force="csr_merge", units=1234) as plan:
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_MERGE_COORDS).reshape(-1, 2),
                              oracle.merge_split(A.rowptr, A.m, 1234))
    B = matrix("block")
    with sd.sd_plan_ex(B, 64, force="bsr") as plan:
        bp, bc, bv = oracle.to_bsr(B, 16)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_BLOCK_PTR), bp)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_BLOCK_COL), bc)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_BLOCK_VAL).view(np.uint32),
                              bv.ravel().view(np.uint32))
    with sd.sd_plan_ex(matrix("laplace"), 64, force="ell") as plan:
        w, ec, ev = oracle.to_ell(matrix("laplace"))
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_ELL_COL), ec.ravel())
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_ELL_VAL).view(np.uint32), ev.ravel().view(np.uint32))
    R = matrix("rmat")
    with sd.sd_plan_ex(R, 64, force="win", window_rows=64, heavy_threshold=100, chunk_nnz=37) as plan:
        light, _ = oracle.heavy_split(R.rowptr, R.m, 100, 37)
        light = oracle.light_by_last_col(R, light)
        lptr, col, val, chunks = oracle.split_layout(R, 100, 37, light)
        wp, wc, code = oracle.split_windows(lptr, col, len(light), 64, (16 << 10) // 256)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_ROWPTR), lptr)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_CHUNKS).reshape(-1, 3), chunks)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_WIN_PTR), wp)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_WIN_COLS), wc)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_WIN_CODE), code)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_WIN_VAL).view(np.uint32), val.view(np.uint32))
    with sd.sd_plan_ex(A, 64, force="sell", sell_sigma=50) as plan:
        perm, sp, sc, sv = oracle.to_sell(A, plan.info["sell_c"], 50)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_SELL_PERM), perm)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_SELL_SLICE_PTR), sp)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_SELL_COL), sc)
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_SELL_VAL).view(np.uint32), sv.view(np.uint32))
    with sd.sd_plan_ex(B, 64, force="bell") as plan:
        w, ec, ev = oracle.to_bell(B, 16)
        assert plan.info["bell_width"] == w
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_BLOCK_COL), ec.ravel())
        assert np.array_equal(sd.sd_plan_export(plan, sd.SD_EXPORT_BLOCK_VAL).view(np.uint32),
                              ev.ravel().view(np.uint32))


@pytest.mark.parametrize("mname", ["laplace", "uniform", "ragged", "block", "rmat"])
@pytest.mark.parametrize("R", [1, 5, 32, 64, 256, 2048])
@pytest.mark.parametrize("n", [8, 64, 100, 256])
def test_window_sizes(mname, R, n):
    """Column windows at forced window sizes: a ragged last window, windows of
    one row (nothing staged), windows larger than a workgroup's row pass, and
    windows whose staged set is capped by the LDS budget (n = 256, R = 2048),
    with heavy rows through chunks."""
    A = matrix(mname)
    B = gen.dense_normal(A.k, n, seed=R)
    C64, S = oracle.spmm(A, B)
    print(f"case win {mname} R={R} n={n}", flush=True)
    with sd.sd_plan_ex(A, n, force="win", window_rows=R, heavy_threshold=200, chunk_nnz=64) as plan:
        assert plan.info["window_rows"] == R
        assert plan.info["window_max"] * 4 * min(n, plan.info["col_tile"]) <= 16 << 10
        for mis in (False, True):
            assert_close(run(sd, plan, B, A.m, misalign=mis), C64, S, f"win/{mname}/{R}/{n}/{mis}")


@pytest.mark.parametrize("fam,opts", [("csr_row", {}), ("ell", {}), ("csr_merge", {"units": 999}),
                                      ("bsr", {"engine": "mfma"}), ("bsr", {"engine": "valu"}), ("win", {}),
                                      ("sell", {})])
@pytest.mark.parametrize("order,chunk", [(1, 0), (2, 0), (3, 2), (3, 5), (3, 64), (3, 100000)])
def test_workgroup_orders(fam, opts, order, chunk):
    """Every workgroup order covers every row exactly once (C starts as NaN)."""
    A = matrix("laplace" if fam in ("ell", "win") else "block" if fam == "bsr" else "ragged")
    n = 64
    B = gen.dense_normal(A.k, n, seed=order * 7 + chunk)
    C64, S = oracle.spmm(A, B)
    print(f"case order {fam} {opts} order={order} chunk={chunk}", flush=True)
    with sd.sd_plan_ex(A, n, force=fam, wg_order=order, wg_chunk=chunk, **opts) as plan:
        assert plan.info["wg_order"] == order
        assert_close(run(sd, plan, B, A.m), C64, S, f"order/{fam}/{order}/{chunk}")


def test_stream_ordering_and_reuse():
    """A plan is reusable across dense operands and honours the caller's stream."""
    A = matrix("laplace")
    n = 64
    s = torch.cuda.Stream()
    with sd.sd_plan(A, n) as plan:
        outs = []
        for seed in range(3):
            B = gen.dense_uniform(A.k, n, seed=seed)
            Bd = torch.from_numpy(B).cuda()
            Cd = torch.empty((A.m, n), device="cuda")
            s.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(s):
                sd.sd_spmm(plan, Bd, Cd, s)
                Cd.record_stream(s)
            outs.append((B, Cd))
        s.synchronize()
        for B, Cd in outs:
            C64, S = oracle.spmm(A, B)
            assert_close(Cd.cpu().numpy(), C64, S, "reuse")


@pytest.mark.parametrize("mname", ["laplace", "rmat", "block", "ragged"])
def test_measured_plan_search(mname):
    """The measured selection returns a correct plan no slower than the
    rule-based one, and a second call is served from the choice cache."""
    A = matrix(mname)
    n = 64
    sd.sd_plan_cache_clear()
    B = gen.dense_normal(A.k, n, seed=21)
    C64, S = oracle.spmm(A, B)
    with sd.sd_plan_ex(A, n, search=True) as plan:
        info = plan.info
        assert info["search_candidates"] >= 2 and info["search_cache_hit"] == 0
        assert info["search_best_ms"] <= info["search_rule_ms"]
        assert_close(run(sd, plan, B, A.m), C64, S, f"search/{mname}")
        chosen = (plan.family, info["engine"], info["heavy_threshold"], info["chunk_nnz"])
    with sd.sd_plan_ex(A, n, search=True) as plan:
        assert plan.info["search_cache_hit"] == 1
        assert (plan.family, plan.info["engine"], plan.info["heavy_threshold"], plan.info["chunk_nnz"]) == chosen
        assert_close(run(sd, plan, B, A.m), C64, S, f"search-cached/{mname}")
    sd.sd_plan_cache_clear()


def assert_same_plan(again: dict, first: dict):
    """What the cache rebuilt is what the search timed.  `reach` is computed under
    the default workgroup order only, and a recorded order is explicit."""
    skip = ("search_cache_hit", "search_candidates", "search_best_ms", "search_rule_ms", "reach")
    assert {f: v for f, v in again.items() if f not in skip} == {f: v for f, v in first.items() if f not in skip}


@pytest.mark.parametrize("mname", ["rmat", "laplace"])
@pytest.mark.parametrize("n", [5, 9, 17, 31])
def test_search_cache_hit_at_odd_widths(mname, n):
    """A choice recorded at a width of no whole 4 columns (rows shared by lane
    groups there) is accepted and rebuilt."""
    A = matrix(mname)
    B = gen.dense_normal(A.k, n, seed=n)
    sd.sd_plan_cache_clear()
    try:
        with sd.sd_plan_ex(A, n, search=True) as first, sd.sd_plan_ex(A, n, search=True) as again:
            assert again.info["search_cache_hit"] == 1
            assert_same_plan(again.info, first.info)
            assert run(sd, again, B, A.m).tobytes() == run(sd, first, B, A.m).tobytes()
    finally:
        sd.sd_plan_cache_clear()


def test_search_keeps_streamed_rows(tmp_path):
    """Ragged rows around a narrow band: the rule streams them, the same rows
    unstreamed in the same workgroup order are another candidate, and the recorded
    choice rebuilds the plan that was timed."""
    rng = np.random.default_rng(3)
    m, n, band = 200003, 64, 820
    lens = rng.integers(8, 41, m)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows = np.repeat(np.arange(m), lens)
    step = band // lens[rows]
    cols = np.clip(rows - band // 2, 0, m - band) + (np.arange(rows.size) - rowptr[rows]) * step
    cols += rng.integers(0, 1 << 30, rows.size) % step
    A = gen.CSR(m, m, rowptr, cols.astype(np.int32), rng.uniform(-1, 1, rows.size).astype(np.float32))
    dev = [torch.from_numpy(x).cuda() for x in (A.rowptr, A.colidx, A.values)]
    opts = dict(force="csr_row")
    with sd.sd_plan_device(*dev, m, m, A.nnz, n, **opts) as rule, \
            sd.sd_plan_device(*dev, m, m, A.nnz, n, wg_order=1, **opts) as plain:
        assert rule.info["stream_rows"] > 0 and rule.info["wg_order"] == 1
        assert plain.info["stream_rows"] == 0 and plain.info["wg_order"] == 1
    with sd.sd_plan_device(*dev, m, m, A.nnz, n) as rule:
        assert rule.family == "csr_row" and rule.info["stream_rows"] > 0
    sd.sd_plan_cache_clear()
    try:
        with sd.sd_plan_device(*dev, m, m, A.nnz, n, search=True) as first:
            info = dict(first.info)
        print(f"search chose {first.family} stream_rows={info['stream_rows']}", flush=True)
        path = tmp_path / "choices.bin"
        sd.sd_plan_cache_save(path)
        with sd.sd_plan_device(*dev, m, m, A.nnz, n, search=True) as again:
            assert again.info["search_cache_hit"] == 1
            assert_same_plan(again.info, info)
        sd.sd_plan_cache_clear()
        sd.sd_plan_cache_load(path)
        with sd.sd_plan_device(*dev, m, m, A.nnz, n, search=True) as loaded:
            assert loaded.info["search_cache_hit"] == 1
            assert_same_plan(loaded.info, info)
    finally:
        sd.sd_plan_cache_clear()


def test_search_choice_saved_and_loaded(tmp_path):
    """A measured choice written to a cache file and loaded into an empty
    cache (as a new process would) is reused without timing: same plan, same
    output bits."""
    A = matrix("ragged")
    n = 32
    sd.sd_plan_cache_clear()
    B = gen.dense_normal(A.k, n, seed=5)
    try:
        with sd.sd_plan_ex(A, n, search=True) as first, \
                sd.sd_plan_ex(A, n, search=True, transpose=True) as first_t:
            info, info_t = dict(first.info), dict(first_t.info)
            C1 = run(sd, first, B, A.m)
        assert sd.sd_plan_cache_size() == 2
        path = tmp_path / "choices.bin"
        sd.sd_plan_cache_save(path)
        sd.sd_plan_cache_clear()
        assert sd.sd_plan_cache_size() == 0
        sd.sd_plan_cache_load(path)
        assert sd.sd_plan_cache_size() == 2
        with sd.sd_plan_ex(A, n, search=True) as again:
            assert again.info["search_cache_hit"] == 1 and again.info["search_candidates"] == 0
            skip = ("search_cache_hit", "search_candidates", "search_best_ms", "search_rule_ms")
            assert {f: v for f, v in again.info.items() if f not in skip} == \
                {f: v for f, v in info.items() if f not in skip}
            assert run(sd, again, B, A.m).tobytes() == C1.tobytes()
        with sd.sd_plan_ex(A, n, search=True, transpose=True) as again_t:
            assert again_t.info["search_cache_hit"] == 1 and again_t.info["family"] == info_t["family"]
        # another width is another key: searched afresh
        with sd.sd_plan_ex(A, 8, search=True) as other:
            assert other.info["search_cache_hit"] == 0
        assert sd.sd_plan_cache_size() == 3
    finally:
        sd.sd_plan_cache_clear()


@pytest.mark.parametrize("fam", ["csr_row", "csr_split", "csr_merge", "ell", "win", "sell"])
@pytest.mark.parametrize("n,col_tile", [(128, 64), (128, 16), (96, 32), (64, 4), (10, 8)])
def test_column_tiles(fam, n, col_tile):
    """The dense width processed in several column passes (K tiles)."""
    A = matrix("rmat")
    B = gen.dense_normal(A.k, n, seed=col_tile)
    C64, S = oracle.spmm(A, B)
    with sd.sd_plan_ex(A, n, force=fam, col_tile=col_tile, heavy_threshold=64, chunk_nnz=64) as plan:
        assert plan.info["col_passes"] == -(-n // plan.info["col_tile"])
        for mis in (False, True):
            assert_close(run(sd, plan, B, A.m, misalign=mis), C64, S, f"coltile/{fam}/{n}/{col_tile}/{mis}")
