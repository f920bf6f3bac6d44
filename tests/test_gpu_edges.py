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
