"""GPU parity at the edges of the kernels' shape ranges (needs an MI355X):
windows that are no multiple of a row tile, lengths around tile, chunk and
segment boundaries, against the fp64 oracle as in test_gpu_parity."""
import pytest

import test_gpu_parity as TP
from oracle import ref
from paper_2606_14782_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    ref.set_threads(16)


def _wl(layers, hq, hkv, d, window, pool, dtype, lens, budgets, seed=31):
    return inputs.Workload("shapes", layers, hq, hkv, d, window, pool, dtype, tuple(lens), tuple(budgets),
                           tuple((0, 0) for _ in lens), 0, seed)


@pytest.mark.parametrize("hq,hkv,d,window,lens", [
    (14, 2, 64, 16, (33, 511, 513, 1025)),     # seven 16-query heads: rows end inside a row tile
    (6, 2, 128, 31, (64, 543, 2048)),          # the last query of a head inside a run of four rows
    (6, 2, 64, 33, (2049, 65)),                # a window one row past a tile, keys one past a segment
    (4, 4, 128, 1, (32, 512, 2080)),           # one-row windows: every row a last query
])
def test_window_rows(hq, hkv, d, window, lens):
    """Windows other than 32 queries: the causal edge and the last-query rows
    fall inside row tiles and inside a lane's runs of four rows."""
    wl = _wl(3, hq, hkv, d, window, 5, "bf16", lens, [max(1, n // 8) for n in lens])
    TP.run_case(f"window-{window}", wl, supplied_lse=True)
