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


@pytest.mark.parametrize("hq,hkv,d,window,dtype,lens", [
    (4, 4, 64, 8, "fp32", (512, 130)),           # one row tile: waves without a tile
    (8, 1, 128, 32, "fp32", (700, 4099)),        # 256 rows of fp32 d 128: the largest LDS
    (28, 4, 128, 32, "bf16", (513, 2049, 97)),   # seven row tiles over the row groups
    (6, 2, 128, 16, "bf16", (8191, 33)),         # two row tiles, two chunks per workgroup
    (5, 1, 64, 20, "bf16", (6145,)),             # rows that end inside the last tile
    (2, 2, 64, 32, "fp32", (1025, 64, 3000)),
])
@pytest.mark.parametrize("wide", [True, False])
def test_small_grids(hq, hkv, d, window, dtype, lens, wide, monkeypatch):
    """Grids that do not fill the GPU: the wide passes (one launch per layer in
    the prompt call) against the oracle, the prompt call against the per-layer
    calls bit for bit, and the same shapes on the passes of larger grids
    (BACON_WIDE=0)."""
    import torch
    import parity as P
    from paper_2606_14782_amd import bacon
    if not wide:
        monkeypatch.setenv("BACON_WIDE", "0")
    wl = _wl(7, hq, hkv, d, window, 7, dtype, lens, [max(1, n // 10) for n in lens])
    TP.run_case(f"small-grid wide={wide}", wl, split=False, supplied_lse=True)
    batch = bacon.BatchLayout(wl.cu_seqlens, wl.budgets_arr)
    xs = [inputs.layer_inputs(wl, l) for l in range(wl.num_layers)]
    qs, ks, vs = ([P.to_dev(x[n], wl) for x in xs] for n in ("q_win", "k", "v"))
    a, b = P.make_ctx(wl), P.make_ctx(wl)
    a.bacon_begin_prompt(batch)
    want = [a.bacon_compress_layer(l, batch, qs[l], ks[l], vs[l]) for l in range(wl.num_layers)]
    b.bacon_begin_prompt(batch)
    got = b.bacon_compress_prompt(0, batch, qs, ks, vs)
    torch.cuda.synchronize()
    for l in range(wl.num_layers):
        for x, y in zip(got[l], want[l]):
            assert torch.equal(x, y), f"layer {l}"
