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
