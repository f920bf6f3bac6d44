"""CPU tests of the native library: the C ABI (symbols and struct layouts
against include/sparseditto.h), the host-side logic against the oracle bit
for bit (analysis, conversions, partitions, transpose) using host-only plans,
error paths, and the footprint model against the paper's worked numbers."""
import ctypes
import json
import os
import re
import subprocess

import numpy as np
import pytest

import gen
import oracle
import paper_2608_05033_amd as sd
from builders import from_rows, nemeth_like, shen_like

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "sparseditto.h")
HOST = sd.PLACEMENT_HOST


def header_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(sd_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_function():
    names = header_functions()
    assert "sd_spmm" in names and "sd_plan_ex" in names
    lib = ctypes.CDLL(sd.LIB_PATH)
    missing = [n for n in names if not hasattr(lib, n)]
    assert not missing, missing
    assert set(names) == set(sd.EXPORTED)


def test_struct_layouts_match_header(tmp_path):
    """Compile a probe against the header and compare every offset with ctypes."""
    structs = {"sd_csr_t": sd.sd_csr_t, "sd_stats_t": sd.sd_stats_t, "sd_plan_opts_t": sd.sd_plan_opts_t,
               "sd_plan_info_t": sd.sd_plan_info_t}
    lines = ['#include <stdio.h>', '#include <stddef.h>', f'#include "{HEADER}"', "int main(void) {"]
    for sname, cls in structs.items():
        lines.append(f'printf("{sname} size %zu\\n", sizeof({sname}));')
        for fname, _ in cls._fields_:
            lines.append(f'printf("{sname} {fname} %zu\\n", offsetof({sname}, {fname}));')
    lines.append("return 0; }")
    src = tmp_path / "probe.c"
    src.write_text("\n".join(lines))
    exe = tmp_path / "probe"
    subprocess.check_call(["gcc", "-o", str(exe), str(src)])
    out = subprocess.check_output([str(exe)]).decode().split("\n")
    for line in filter(None, out):
        sname, fname, val = line.split()
        cls = structs[sname]
        if fname == "size":
            assert ctypes.sizeof(cls) == int(val), sname
        else:
            assert getattr(cls, fname).offset == int(val), (sname, fname)


def ragged(m, k, seed):
    rng = np.random.default_rng(seed)
    r = rng.integers(0, 50, m)
    r[rng.random(m) < 0.2] = 0
    if m > 5:
        r[m // 2] = k
    return np.minimum(r, k)


def torch_has_gpu():
    try:
        import torch
        return torch.cuda.is_available()
    except Exception:  # pragma: no cover
        return False


MATS = {
    "ragged": lambda: gen.random_rows(700, 900, ragged(700, 900, 1), seed=1),
    "rmat": lambda: gen.rmat(12, 50000, seed=2),
    "block": lambda: gen.block(40, 45, 16, 9, 12, 0.9, 3),
    "laplace": lambda: gen.laplacian3d(9, 7, 5),
    "uniform": lambda: gen.uniform_rows(300, 500, 8, 4),
    "empty": lambda: gen.random_rows(50, 30, np.zeros(50, np.int32), seed=5),
    "onerow": lambda: gen.random_rows(1, 4000, np.array([4000], np.int32), seed=6),
    "shen": shen_like,
}


@pytest.mark.parametrize("name", list(MATS))
def test_analyze_matches_oracle_bitwise(name):
    A = MATS[name]()
    for thr in (128, 1, 200):
        st = sd.sd_analyze(A, dense_threshold=thr)
        ref = oracle.stats(A, dense_threshold=thr)
        for key, v in ref.items():
            if isinstance(v, np.ndarray):
                assert np.array_equal(st[key], v), key
            elif isinstance(v, float):
                assert np.float64(st[key]).tobytes() == np.float64(v).tobytes(), (key, st[key], v)
            else:
                assert st[key] == v, key


@pytest.mark.parametrize("name", ["ragged", "rmat", "uniform", "empty", "onerow"])
@pytest.mark.parametrize("T,c", [(1, 1), (4, 3), (32, 32), (256, 256), (10**6, 7)])
def test_chunk_order_matches_oracle(name, T, c):
    """The chunk processing order: by middle column (the default) as the
    oracle defines it over the split layout, or the chunk list itself."""
    A = MATS[name]()
    light, _ = oracle.heavy_split(A.rowptr, A.m, T, c)
    _, col, _, chunks = oracle.split_layout(A, T, c, oracle.light_by_last_col(A, light))
    for order, want in (("auto", oracle.chunks_by_mid_col(col, chunks)),
                        ("mid_col", oracle.chunks_by_mid_col(col, chunks)),
                        ("list", np.arange(len(chunks), dtype=np.int32))):
        with sd.sd_plan_ex(A, 8, force="csr_split", heavy_threshold=T, chunk_nnz=c, chunk_order=order,
                           placement=HOST) as p:
            assert p.info["chunk_order"] == (1 if order == "list" else 2)
            assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_CHUNK_ORDER), want)
    with pytest.raises(sd.SparseDittoError):
        sd.sd_plan_ex(A, 8, force="csr_split", chunk_order=3, placement=HOST)


@pytest.mark.parametrize("name", ["ragged", "rmat", "uniform", "empty", "onerow"])
@pytest.mark.parametrize("T,c", [(1, 1), (4, 3), (32, 32), (256, 256), (10**6, 7)])
def test_heavy_split_matches_oracle(name, T, c):
    """Light rows by last column (the default) and ascending, and the chunks."""
    A = MATS[name]()
    light, chunks = oracle.heavy_split(A.rowptr, A.m, T, c)
    for order, want in (("auto", oracle.light_by_last_col(A, light)), ("last_col", oracle.light_by_last_col(A, light)),
                        ("ascending", light)):
        with sd.sd_plan_ex(A, 8, force="csr_split", heavy_threshold=T, chunk_nnz=c, light_order=order,
                           placement=HOST) as p:
            assert p.info["light_order"] == (1 if order == "ascending" else 2)
            assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_LIGHT_ROWS), want)
            # the split layout: light rows in list order, then heavy rows; chunks in its coordinates
            lptr, col, val, lchunks = oracle.split_layout(A, T, c, want)
            assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_CHUNKS).reshape(-1, 3), lchunks)
            assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_ROWPTR), lptr)
            assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_COLIDX), col)
            assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_VALUES).view(np.uint32), val.view(np.uint32))
            assert np.array_equal(lchunks[:, 0], chunks[:, 0])
            assert np.array_equal(lchunks[:, 2] - lchunks[:, 1], chunks[:, 2] - chunks[:, 1])
            assert p.info["n_chunks"] == len(chunks) and p.info["n_light"] == len(light)
    with pytest.raises(sd.SparseDittoError) as e:
        sd.sd_plan_ex(A, 8, force="csr_split", light_order=3, placement=HOST)
    assert e.value.status == sd.SD_ERR_INVALID_VALUE


@pytest.mark.parametrize("name", ["ragged", "rmat", "uniform", "empty", "onerow", "laplace"])
@pytest.mark.parametrize("U", [1, 2, 3, 17, 1000, 100000])
def test_merge_split_matches_oracle(name, U):
    A = MATS[name]()
    with sd.sd_plan_ex(A, 8, force="csr_merge", units=U, placement=HOST) as p:
        got = sd.sd_plan_export(p, sd.SD_EXPORT_MERGE_COORDS).reshape(-1, 2)
        assert np.array_equal(got, oracle.merge_split(A.rowptr, A.m, U))


@pytest.mark.parametrize("name", ["ragged", "rmat", "block", "laplace", "empty", "onerow"])
def test_block_conversions_match_oracle(name):
    A = MATS[name]()
    with sd.sd_plan_ex(A, 64, force="bsr", placement=HOST) as p:
        bp, bc, bv = oracle.to_bsr(A, 16)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_BLOCK_PTR), bp)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_BLOCK_COL), bc)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_BLOCK_VAL).view(np.uint32), bv.ravel().view(np.uint32))
    with sd.sd_plan_ex(A, 64, force="bell", placement=HOST) as p:
        w, ec, ev = oracle.to_bell(A, 16)
        assert p.info["bell_width"] == w
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_BLOCK_COL), ec.ravel())
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_BLOCK_VAL).view(np.uint32), ev.ravel().view(np.uint32))


@pytest.mark.parametrize("name", ["ragged", "rmat", "laplace", "uniform", "empty", "onerow"])
def test_ell_conversion_matches_oracle(name):
    A = MATS[name]()
    with sd.sd_plan_ex(A, 16, force="ell", placement=HOST) as p:
        w, ec, ev = oracle.to_ell(A)
        assert p.info["ell_width"] == w and p.info["m_rep"] == 8 * A.m * w
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_ELL_COL), ec.ravel())
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_ELL_VAL).view(np.uint32), ev.ravel().view(np.uint32))


@pytest.mark.parametrize("name", ["ragged", "rmat", "laplace", "uniform", "block", "empty", "onerow"])
@pytest.mark.parametrize("R,T,c", [(1, 512, 2048), (16, 40, 17), (64, 10**6, 7), (128, 256, 128), (512, 30, 64)])
@pytest.mark.parametrize("n", [16, 256])
def test_window_conversion_matches_oracle(name, R, T, c, n):
    """Packed column windows over the split layout: the split arrays, the
    window pointers, staged columns and entry codes equal the oracle's, with
    the staged set capped to the columns that fit 16 KiB of LDS (n floats per
    staged column: 64 B at n = 16, 1 KiB at n = 256)."""
    A = MATS[name]()
    cap = (16 << 10) // (4 * n)
    light, _ = oracle.heavy_split(A.rowptr, A.m, T, c)
    light = oracle.light_by_last_col(A, light)
    lptr, col, val, chunks = oracle.split_layout(A, T, c, light)
    wp, wc, code = oracle.split_windows(lptr, col, len(light), R, cap)
    with sd.sd_plan_ex(A, n, force="win", window_rows=R, heavy_threshold=T, chunk_nnz=c, placement=HOST) as p:
        info = p.info
        assert info["window_rows"] == R and info["heavy_threshold"] == T and info["chunk_nnz"] == c
        assert info["window_staged"] == wc.size
        assert info["window_max"] == (int(np.diff(wp).max()) if wp.size > 1 else 0)
        assert info["window_staged_uses"] == int((code <= -2).sum())
        nw = wp.size - 1
        assert info["m_rep"] == 8 * A.nnz + 4 * (A.m + 1) + 4 * info["n_light"] + 16 * info["n_chunks"] + \
            4 * info["n_heavy"] + 4 * (info["n_heavy"] + 1) + 4 * (nw + 1) + 4 * wc.size
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_LIGHT_ROWS), light)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_ROWPTR), lptr)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_CHUNKS).reshape(-1, 3), chunks)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_CHUNK_ORDER), oracle.chunks_by_mid_col(col, chunks))
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_WIN_PTR), wp)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_WIN_COLS), wc)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_WIN_CODE), code)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_WIN_VAL).view(np.uint32), val.view(np.uint32))
        for what in (sd.SD_EXPORT_ELL_COL, sd.SD_EXPORT_COLIDX):
            with pytest.raises(sd.SparseDittoError):
                sd.sd_plan_export(p, what)


@pytest.mark.parametrize("name", ["ragged", "rmat", "laplace", "uniform", "block", "empty", "onerow"])
@pytest.mark.parametrize("n,sigma", [(64, 0), (64, 1), (8, 100), (256, 7), (1, 1000000)])
def test_sell_conversion_matches_oracle(name, n, sigma):
    A = MATS[name]()
    with sd.sd_plan_ex(A, n, force="sell", sell_sigma=sigma, placement=HOST) as p:
        info = p.info
        C = info["sell_c"]
        assert C == 64 // info["lanes_per_row"]
        assert info["sell_sigma"] == (sigma if sigma > 0 else 8 * C)
        perm, sp, col, val = oracle.to_sell(A, C, info["sell_sigma"])
        assert info["sell_slices"] == sp.size - 1 and info["sell_slots"] == sp[-1]
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_SELL_PERM), perm)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_SELL_SLICE_PTR), sp)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_SELL_COL), col)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_SELL_VAL).view(np.uint32), val.view(np.uint32))


def test_window_staged_set_capped_by_lds():
    """A window stages at most the columns that fit 16 KiB of LDS (16 at
    n = 256, 1 KiB each), keeping its most used; every window size is
    accepted, and a negative one is refused."""
    A = MATS["block"]()  # 16x16 blocks: a window shares its block-rows' columns
    with sd.sd_plan_ex(A, 256, force="win", window_rows=256, placement=HOST) as p:
        assert 0 < p.info["window_max"] <= 16
    with sd.sd_plan_ex(A, 256, force="win", window_rows=4096, placement=HOST) as p:
        assert p.info["window_max"] == 16
    with pytest.raises(sd.SparseDittoError) as e:
        sd.sd_plan_ex(A, 256, force="win", window_rows=-1, placement=HOST)
    assert e.value.status == sd.SD_ERR_INVALID_VALUE


@pytest.mark.parametrize("name", ["ragged", "rmat", "laplace", "empty", "onerow"])
def test_transpose_matches_oracle(name):
    A = MATS[name]()
    with sd.sd_plan_ex(A, 4, force="csr_row", transpose=True, placement=HOST) as p:
        tr, tc, tv = oracle.transpose(A)
        assert p.info["m"] == A.k and p.info["k"] == A.m
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_ROWPTR), tr)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_COLIDX), tc)
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_VALUES).view(np.uint32), tv.view(np.uint32))


def test_csr_copy_is_bitwise():
    A = MATS["ragged"]()
    A.values[:5] = [np.nan, -0.0, np.inf, 1e-45, -np.inf]
    with sd.sd_plan_ex(A, 4, force="csr_row", placement=HOST) as p:
        assert np.array_equal(sd.sd_plan_export(p, sd.SD_EXPORT_VALUES).view(np.uint32), A.values.view(np.uint32))


# ----------------------------------------------------------- error paths ---

def _bad(rowptr, colidx, m, k):
    return dict(rowptr=np.array(rowptr, np.int32), colidx=np.array(colidx, np.int32),
                values=np.ones(len(colidx), np.float32), m=m, k=k)


@pytest.mark.parametrize("case", [
    _bad([1, 2], [0], 1, 3),            # rowptr[0] != 0
    _bad([0, 2, 1], [0, 1], 2, 3),      # decreasing rowptr
    _bad([0, 1], [3], 1, 3),            # column out of range
    _bad([0, 1], [-1], 1, 3),           # negative column
    _bad([0, 2], [1, 1], 1, 3),         # duplicate column
    _bad([0, 2], [2, 1], 1, 3),         # unsorted columns
])
def test_invalid_csr_rejected(case):
    with pytest.raises(sd.SparseDittoError) as e:
        sd.sd_analyze(**case)
    assert e.value.status == sd.SD_ERR_INVALID_CSR
    with pytest.raises(sd.SparseDittoError) as e:
        sd.sd_plan_ex(n=4, placement=HOST, **case)
    assert e.value.status == sd.SD_ERR_INVALID_CSR


def test_rowptr_end_must_equal_nnz():
    c = sd.sd_csr_t(2, 3, 5, None, None, None)  # rowptr missing
    st = sd.sd_stats_t()
    assert sd._lib.sd_analyze(ctypes.byref(c), 0, ctypes.byref(st)) == sd.SD_ERR_INVALID_VALUE
    rp = np.array([0, 1, 2], np.int32)
    ci = np.array([0, 1], np.int32)
    vv = np.ones(2, np.float32)
    c = sd.sd_csr_t(2, 3, 3, rp.ctypes.data, ci.ctypes.data, vv.ctypes.data)  # nnz says 3, rowptr[m] = 2
    assert sd._lib.sd_analyze(ctypes.byref(c), 0, ctypes.byref(st)) == sd.SD_ERR_INVALID_CSR
    c = sd.sd_csr_t(2, 3, 1 << 31, rp.ctypes.data, ci.ctypes.data, vv.ctypes.data)
    assert sd._lib.sd_analyze(ctypes.byref(c), 0, ctypes.byref(st)) == sd.SD_ERR_OVERFLOW


def test_invalid_arguments():
    A = MATS["uniform"]()
    for kw in [dict(n=0), dict(n=-3), dict(n=4, force=9), dict(n=4, rows_per_group=3), dict(n=4, gather_unroll=5),
               dict(n=4, engine=7), dict(n=4, placement=5), dict(n=4, units=-1)]:
        n = kw.pop("n")
        with pytest.raises(sd.SparseDittoError) as e:
            sd.sd_plan_ex(A, n, **({"placement": HOST} | kw))
        assert e.value.status == sd.SD_ERR_INVALID_VALUE, kw
    with pytest.raises(sd.SparseDittoError) as e:
        sd.sd_analyze(A, dense_threshold=300)
    assert e.value.status == sd.SD_ERR_INVALID_VALUE
    assert sd._lib.sd_plan(None, 4, None) == sd.SD_ERR_INVALID_VALUE
    assert sd._lib.sd_spmm(None, None, None, None) == sd.SD_ERR_INVALID_VALUE
    sd._lib.sd_plan_destroy(None)  # no-op


def test_block_engine_choice():
    """MFMA serves every width (partial column tiles); VALU only when forced."""
    A = MATS["block"]()
    for n in (1, 3, 8, 16, 40, 50, 64, 100):
        with sd.sd_plan_ex(A, n, force="bsr", placement=HOST) as p:
            assert p.info["engine"] == sd.SD_ENGINE_MFMA
        with sd.sd_plan_ex(A, n, force="bsr", engine="valu", placement=HOST) as p:
            assert p.info["engine"] == sd.SD_ENGINE_VALU


def _lanes(n):
    """Lanes per row covering a width of n floats (four columns per lane from n = 4 on)."""
    lanes = -(-n // 4) if n >= 4 else n
    g = 1
    while g < lanes and g < 64:
        g *= 2
    return g


@pytest.mark.parametrize("fam", ["csr_row", "csr_split"])
@pytest.mark.parametrize("n", [1, 3, 8, 32, 64])
@pytest.mark.parametrize("S", [1, 2, 8, 64])
def test_row_slices_option(fam, n, S):
    """Slices need G <= 8 and G * S <= 64; the plan reports G * S lanes per row."""
    A = MATS["uniform"]()
    G = _lanes(n)
    if S > 1 and (G > 8 or G * S > 64):
        with pytest.raises(sd.SparseDittoError) as e:
            sd.sd_plan_ex(A, n, force=fam, row_slices=S, placement=HOST)
        assert e.value.status == sd.SD_ERR_UNSUPPORTED
        return
    with sd.sd_plan_ex(A, n, force=fam, row_slices=S, placement=HOST) as p:
        assert p.info["row_slices"] == S
        assert p.info["lanes_per_row"] == G * S
        if S > 1:
            assert p.info["rows_per_group"] == 1


@pytest.mark.parametrize("fam", ["csr_row", "csr_split"])
@pytest.mark.parametrize("n", [1, 2, 3, 5, 9, 10, 13, 17, 30, 31, 32, 33, 64])
def test_planned_values_are_accepted_as_options(fam, n):
    """A plan's own slice count and split sizes, passed back as options (as the
    search's recorded choices are), give the same plan at every width."""
    A = MATS["rmat"]()
    with sd.sd_plan_ex(A, n, force=fam, placement=HOST) as p:
        first = dict(p.info)
    back = dict(row_slices=first["row_slices"])
    if fam == "csr_split":
        assert first["row_slices"] > 1 or n > 32
        back.update(heavy_threshold=first["heavy_threshold"], chunk_nnz=first["chunk_nnz"])
    with sd.sd_plan_ex(A, n, force=fam, placement=HOST, **back) as p:
        assert p.info == first


def test_row_slices_invalid_and_other_families():
    A = MATS["uniform"]()
    for bad in (-1, 3, 6, 128):
        with pytest.raises(sd.SparseDittoError) as e:
            sd.sd_plan_ex(A, 8, force="csr_row", row_slices=bad, placement=HOST)
        assert e.value.status == sd.SD_ERR_INVALID_VALUE
    for fam in ("ell", "csr_merge", "sell"):  # not a sliced family: the option is ignored
        with sd.sd_plan_ex(A, 8, force=fam, row_slices=4, placement=HOST) as p:
            assert p.info["row_slices"] == 0


@pytest.mark.skipif(torch_has_gpu(), reason="a GPU is visible")
def test_device_analysis_needs_a_device():
    with pytest.raises(sd.SparseDittoError) as e:
        sd.sd_analyze_device(0, 0, 0, 4, 4, 0)
    assert e.value.status == sd.SD_ERR_NO_DEVICE


def test_device_plan_argument_checks():
    """Checked before any device pointer is read (the pointers here are never dereferenced)."""
    for kw, status in ((dict(rowptr=0), sd.SD_ERR_INVALID_VALUE), (dict(n=0), sd.SD_ERR_INVALID_VALUE),
                       (dict(m=-1), sd.SD_ERR_INVALID_CSR), (dict(colidx=0), sd.SD_ERR_INVALID_VALUE),
                       (dict(wg_order=9), sd.SD_ERR_INVALID_VALUE), (dict(rows_per_group=3), sd.SD_ERR_INVALID_VALUE)):
        args = dict(rowptr=256, colidx=512, values=768, m=4, k=4, nnz=3, n=8)
        args.update(kw)
        with pytest.raises(sd.SparseDittoError) as e:
            sd.sd_plan_device(**args)
        assert e.value.status == status, kw


@pytest.mark.skipif(torch_has_gpu(), reason="a GPU is visible")
def test_device_plan_needs_a_device():
    with pytest.raises(sd.SparseDittoError) as e:
        sd.sd_plan_device(256, 512, 768, 4, 4, 3, 8)
    assert e.value.status == sd.SD_ERR_NO_DEVICE


def test_search_needs_a_device():
    with pytest.raises(sd.SparseDittoError) as e:
        sd.sd_plan_ex(MATS["uniform"](), 8, search=True, placement=HOST)
    assert e.value.status == sd.SD_ERR_NO_DEVICE


def test_host_only_plan_refuses_spmm():
    A = MATS["uniform"]()
    with sd.sd_plan_ex(A, 8, placement=HOST) as p:
        with pytest.raises(sd.SparseDittoError) as e:
            sd.sd_spmm(p, 0, 0)
        assert e.value.status == sd.SD_ERR_NO_DEVICE
        assert p.info["device"] == -1 and p.info["legal"] == 1


def test_export_rejects_wrong_kind_and_short_buffer():
    A = MATS["uniform"]()
    with sd.sd_plan_ex(A, 8, force="csr_row", placement=HOST) as p:
        size = ctypes.c_size_t()
        assert sd._lib.sd_plan_export_size(p.handle, sd.SD_EXPORT_CHUNKS, ctypes.byref(size)) == sd.SD_ERR_INVALID_VALUE
        buf = np.empty(4, np.int32)
        assert sd._lib.sd_plan_export(p.handle, sd.SD_EXPORT_ROWPTR, buf.ctypes.data, 16) == sd.SD_ERR_INVALID_VALUE


def test_status_strings():
    for st in range(8):
        assert sd.sd_status_string(st).startswith("SD_")
    assert sd.sd_status_string(99) == "unknown sd_status"


# ------------------------------------------------------- footprint model ---

def _golden():
    with open(os.path.join(ROOT, "tests", "golden", "worked_examples.json")) as f:
        return json.load(f)


def test_footprint_paper_worked_example_shen():
    """CSR footprint 8 nnz + 4 (m + 1) = 4,497,624 B (4.29 MiB) for the
    Shen/e40r0100 counts, Eq. representation-footprint."""
    g = _golden()["shen_e40r0100"]
    with sd.sd_plan_ex(shen_like(), 8, force="csr_row", placement=HOST) as p:
        assert p.info["m_rep"] == g["csr_bytes"]
        assert p.info["m_rep"] / 2 ** 20 == pytest.approx(g["csr_megabytes"]["approx"], abs=g["csr_megabytes"]["tol"])


def test_footprint_paper_worked_example_nemeth():
    """CSR working set including B and C at K = 8: 12.15 MiB for the nemeth26
    counts, Eq. candidate-working-set (M_T = M_rep + W + D_R + D_S)."""
    g = _golden()["nemeth26"]
    with sd.sd_plan_ex(nemeth_like(), g["n"], force="csr_row", placement=HOST) as p:
        info = p.info
        assert info["workspace"] == 0
        assert info["m_t"] == info["m_rep"] + info["d_r"] + info["d_s"]
        assert info["m_t"] / 2 ** 20 == pytest.approx(g["csr_working_set_mib"]["approx"],
                                                     abs=g["csr_working_set_mib"]["tol"])


def test_footprint_components():
    A = MATS["rmat"]()
    n = 32
    with sd.sd_plan_ex(A, n, force="csr_split", heavy_threshold=20, chunk_nnz=16, placement=HOST) as p:
        i = p.info
        assert i["workspace"] == 4 * n * i["n_chunks"]
        # chunk triples and the chunk processing order: 16 bytes per chunk
        assert i["m_rep"] == 8 * A.nnz + 4 * (A.m + 1) + 4 * i["n_light"] + 16 * i["n_chunks"] + 4 * i["n_heavy"] + \
            4 * (i["n_heavy"] + 1)
        assert i["compulsory_bytes"] == 8 * A.nnz + 4 * (A.m + 1) + 4 * A.k * n + 4 * A.m * n
        assert i["q_t"] == pytest.approx(i["m_t"] / i["l2_bytes"])
    B = MATS["block"]()
    with sd.sd_plan_ex(B, 64, force="bsr", placement=HOST) as p:
        i = p.info
        assert i["m_rep"] == 1024 * i["nnzb"] + 4 * i["nnzb"] + 4 * (i["block_rows"] + 1)


def test_planner_rules():
    """The family rules (a heuristic reading; parity unpinned): block formats
    when 16x16 tiles are nearly full, ELL for near-uniform short rows,
    heavy-row split when some row reaches 512 nonzeros (rows from 128 cut into
    chunks of 64, or of 128 at narrow widths, run by middle column), CSR rows
    otherwise."""
    with sd.sd_plan_ex(gen.block(40, 45, 16, 9, 12, 0.97, 3), 64, placement=HOST) as p:
        assert p.family == "bsr" and p.info["engine"] == sd.SD_ENGINE_MFMA
    with sd.sd_plan_ex(MATS["rmat"](), 64, placement=HOST) as p:
        assert p.family == "csr_split" and p.info["heavy_threshold"] == 128 and p.info["chunk_nnz"] == 64
        assert p.info["chunk_order"] == 2 and p.info["light_order"] == 2
    with sd.sd_plan_ex(MATS["rmat"](), 8, placement=HOST) as p:
        assert p.family == "csr_split" and p.info["heavy_threshold"] == 128 and p.info["chunk_nnz"] == 128
    with sd.sd_plan_ex(MATS["laplace"](), 64, placement=HOST) as p:
        assert p.family == "ell" and p.info["ell_width"] == 7
    with sd.sd_plan_ex(MATS["ragged"](), 64, placement=HOST) as p:
        assert p.family == "csr_split"
    with sd.sd_plan_ex(gen.random_rows(500, 400, np.arange(500) % 40, seed=9), 64, placement=HOST) as p:
        assert p.family == "csr_row"


def test_planner_lane_width():
    """Lanes per row at widths of no whole 4 columns (a heuristic reading, set by
    measurement; parity unpinned): four columns per lane where there are waves enough,
    one where rows are few, long or reach over much of B.  The plan describes the lanes
    that it launches with."""
    def lanes(A, n, **kw):
        with sd.sd_plan_ex(A, n, placement=HOST, **kw) as p:
            S = max(1, p.info["row_slices"])
            G = p.info["lanes_per_row"] // S
            assert p.info["col_tile"] in (G, 4 * G) and p.info["col_passes"] == -(-n // p.info["col_tile"])
            return G

    rng = np.random.default_rng(0)
    few = gen.random_rows(3000, 3000, rng.integers(30, 80, 3000), seed=1)
    many = gen.random_rows(100000, 400, rng.integers(2, 12, 100000), seed=1)
    for n, one, four in ((5, 8, 2), (15, 16, 4), (27, 32, 8), (63, 64, 16)):
        assert lanes(few, n, force="csr_row", row_slices=1) == one, n
        if n > 16:
            assert lanes(few, n, force="csr_row") == one and lanes(many, n, force="csr_row") == four, n
        else:  # rows shared by lane groups
            assert lanes(few, n, force="csr_row") == four, n
        assert lanes(few, n, force="csr_row", row_slices=2 if n < 32 else 1) == (four if n < 32 else one), n
    lap = gen.laplacian3d(30, 30, 30)
    wide = gen.uniform_rows(2000, 200000, 24, 0)
    assert [lanes(lap, n, force="ell") for n in (5, 13, 17, 31)] == [2, 4, 8, 8]
    assert [lanes(wide, n, force="ell") for n in (5, 13, 17, 31)] == [8, 16, 32, 32]
    assert [lanes(wide, n, force="ell") for n in (4, 12, 32, 33, 101)] == [1, 4, 8, 16, 32]
    assert [lanes(few, n, force="sell") for n in (7, 31, 101)] == [8, 32, 32]
    assert [lanes(few, n, force="win") for n in (7, 9)] == [8, 4]
    assert [lanes(few, n, force="bsr", engine="valu") for n in (7, 9)] == [8, 4]
    assert [lanes(few, n, force="csr_merge") for n in (7, 31, 47, 101, 150)] == [8, 32, 64, 64, 64]


def test_planner_streamed_rows():
    """Which CSR_ROW plans stream their rows (a heuristic reading, set by measurement;
    parity unpinned): rows around a band whose stretch of B fits, workgroups enough;
    long rows less and later; never under an explicit order, batch or width of 4 or less."""
    def stream(A, n, **kw):
        with sd.sd_plan_ex(A, n, force="csr_row", placement=HOST, **kw) as p:
            assert p.info["wg_order"] == 1 or p.info["stream_rows"] == 0 or kw
            return p.info["stream_rows"]

    def band(m, mean, width):
        lens = np.random.default_rng(m).integers(mean // 2, mean + mean // 2 + 1, m)
        rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        rows = np.repeat(np.arange(m), lens)
        step = width // lens[rows]
        cols = np.clip(rows - width // 2, 0, m - width) + (np.arange(rows.size) - rowptr[rows]) * step
        return gen.CSR(m, m, rowptr, cols.astype(np.int32), np.ones(cols.size, np.float32))

    A = band(100000, 12, 2000)
    assert stream(A, 64) == 2 and stream(A, 128) == 2 and stream(A, 256) == 4 and stream(A, 16) == 0
    for kw in (dict(wg_order=2), dict(wg_order=1), dict(rows_per_group=1), dict(gather_unroll=8)):
        assert stream(A, 64, **kw) == 0
    assert stream(band(100000, 12, 20000), 64) == 0      # wider than the rows of one XCD
    assert stream(band(30000, 12, 1200), 96) == 2 and stream(band(30000, 100, 1200), 96) == 0  # 1,875 workgroups
    assert stream(band(18000, 24, 1200), 180) == 2 and stream(band(18000, 54, 1200), 180) == 0
    assert stream(band(60000, 24, 7000), 256) == 2 and stream(band(60000, 100, 7000), 256) == 0  # 6.8 MiB


def test_planner_slices_at_narrow_widths():
    """Narrow widths (a heuristic reading, set by measurement; parity unpinned):
    heavy-split light rows get 8 lanes (16 at G = 8), the row kernel about one
    round of 4 nonzeros per slice, and N = 1 takes sliced CSR rows instead of ELL."""
    rm = MATS["rmat"]()
    for n, S in ((1, 8), (8, 4), (16, 2), (32, 2), (64, 1), (128, 1)):
        with sd.sd_plan_ex(rm, n, placement=HOST) as p:
            assert p.family == "csr_split" and p.info["row_slices"] == S, (n, p.info["row_slices"])
    lap = MATS["laplace"]()  # 7 nonzeros per interior row: 2 slices of 4
    with sd.sd_plan_ex(lap, 1, placement=HOST) as p:
        assert p.family == "csr_row" and p.info["row_slices"] == 2 and p.info["lanes_per_row"] == 2
    for n in (4, 8, 64):
        with sd.sd_plan_ex(lap, n, placement=HOST) as p:
            assert p.family == "ell" and p.info["row_slices"] == 0
    with sd.sd_plan_ex(lap, 32, force="csr_row", placement=HOST) as p:  # G = 8: one group per row
        assert p.info["row_slices"] == 1
    long_rows = gen.random_rows(500, 400, np.full(500, 100), seed=9)
    with sd.sd_plan_ex(long_rows, 1, force="csr_row", placement=HOST) as p:  # capped at 8 lanes
        assert p.info["row_slices"] == 8


def test_product_does_not_touch_the_oracle():
    """The library and its binding never import or link the test oracle or
    the input generators."""
    pkg = os.path.join(ROOT, "paper_2608_05033_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".cpp", ".hip", ".h")):
                text = open(os.path.join(dirpath, f)).read()
                assert not re.search(r"\b(import|from)\s+(oracle|gen)\b", text), f
                assert "oracle/" not in text and "liboracle" not in text, f
    out = subprocess.check_output(["ldd", sd.LIB_PATH]).decode()
    assert "oracle" not in out and "sdgen" not in out


def _cache_file(records, tag=b"SDPLANC2", rec_size=None, trailing=b""):
    """A cache file in the documented layout: tag, u32 record size, u32 zero,
    u64 count, then (u64 key, sd_plan_opts_t) records."""
    import struct
    rec_size = ctypes.sizeof(sd.sd_plan_opts_t) if rec_size is None else rec_size
    out = tag + struct.pack("<IIQ", rec_size, 0, len(records))
    for key, opts in records:
        out += struct.pack("<Q", key) + bytes(opts)
    return out + trailing


def test_plan_cache_file_round_trip(tmp_path):
    sd.sd_plan_cache_clear()
    empty = tmp_path / "empty.bin"
    sd.sd_plan_cache_save(empty)
    assert empty.read_bytes() == _cache_file([])
    o1 = sd._plan_opts(force="ell", wg_order="chunked", wg_chunk=32)
    o2 = sd._plan_opts(force="csr_split", heavy_threshold=256, chunk_nnz=256)
    src = tmp_path / "two.bin"
    src.write_bytes(_cache_file([(7, o1), (3, o2)]))
    try:
        sd.sd_plan_cache_load(src)
        assert sd.sd_plan_cache_size() == 2
        sd.sd_plan_cache_load(src)  # same keys: replaced, not added
        assert sd.sd_plan_cache_size() == 2
        again = tmp_path / "again.bin"
        sd.sd_plan_cache_save(again)
        assert again.read_bytes() == _cache_file([(3, o2), (7, o1)])  # keys ascending
    finally:
        sd.sd_plan_cache_clear()
    assert sd.sd_plan_cache_size() == 0


@pytest.mark.parametrize("bad", ["tag", "record_size", "truncated", "trailing", "search_record", "auto_record",
                                 "bad_option", "missing"])
def test_plan_cache_load_rejects(tmp_path, bad):
    sd.sd_plan_cache_clear()
    good = sd._plan_opts(force="csr_row")
    body = {
        "tag": _cache_file([(1, good)], tag=b"SDPLANC1"),
        "record_size": _cache_file([(1, good)], rec_size=ctypes.sizeof(sd.sd_plan_opts_t) + 4),
        "truncated": _cache_file([(1, good)])[:-3],
        "trailing": _cache_file([(1, good)], trailing=b"\0"),
        "search_record": _cache_file([(1, good), (2, sd._plan_opts(force="csr_row", search=True))]),
        "auto_record": _cache_file([(1, sd._plan_opts())]),
        "bad_option": _cache_file([(1, sd._plan_opts(force="ell", rows_per_group=3))]),
    }.get(bad)
    path = tmp_path / "c.bin"
    if body is not None:
        path.write_bytes(body)
    with pytest.raises(sd.SparseDittoError) as e:
        sd.sd_plan_cache_load(path)
    assert e.value.status == sd.SD_ERR_IO
    assert sd.sd_plan_cache_size() == 0  # nothing added from a rejected file


def test_plan_cache_null_arguments(tmp_path):
    assert sd._lib.sd_plan_cache_save(None) == sd.SD_ERR_INVALID_VALUE
    assert sd._lib.sd_plan_cache_load(None) == sd.SD_ERR_INVALID_VALUE
    assert sd._lib.sd_plan_cache_size(None) == sd.SD_ERR_INVALID_VALUE
    with pytest.raises(sd.SparseDittoError) as e:
        sd.sd_plan_cache_save(tmp_path / "no_such_dir" / "c.bin")
    assert e.value.status == sd.SD_ERR_IO
