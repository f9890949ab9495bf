"""Host-side checks of bench.py's accounting (no GPU): the roofline counts a
layer's K once (K + Q_win + E written for the launch that completes a
layer's K pass), the launches of a layer add up to the per-layer
algorithmic bytes, combined launches are the sums of their jobs, and the
counter map names every kernel."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_2606_14782_amd import counters, inputs  # noqa: E402

PROMPT_KERNELS = ["window_lse_kr", "lse_merge", "window_score_calib_kr",
                  "window_score_calib_lse_kr", "window_score_calib_lse", "window_score_single",
                  "window_lse_wide", "window_score_calib_wide", "segment_calib", "segment_score",
                  "segment_cand", "final_topk", "segment_select", "layer_stages"]


@pytest.mark.parametrize("name", PROMPT_KERNELS)
def test_kernels_of_the_measured_path_are_accounted(name):
    wl = inputs.workload(3)
    kb, db = bench.kernel_bytes(name, wl), bench.design_bytes(name, wl)
    if name in bench.DESIGN_ONLY:
        assert kb == 0.0
    else:
        assert kb > 0
    assert db >= kb


def test_score_pass_counts_one_layer_of_k():
    """The dual launch (pass 2 of layer l, pass 1 of l+1) completes one layer's
    K pass: K once, Q_win and E written -- 68,419,584 bytes on the 32K video
    workload, 0.24 of 8 TB/s at 35.40 us; its design bytes read K twice."""
    wl = inputs.workload(3)
    K = 32768 * 8 * 128 * 2
    Q = 32 * 32 * 128 * 2
    vec = 32768 * 8 * 4
    for name in bench.SCORE_PASSES:
        assert bench.kernel_bytes(name, wl) == K + Q + vec
    assert bench.kernel_bytes("window_score_calib_lse_kr", wl) == 68419584
    assert bench.design_bytes("window_score_calib_lse_kr", wl) == 2 * (K + Q) + 2 * vec
    frac = 68419584 / 35.40e-6 / 8e12
    assert frac == pytest.approx(0.2416, abs=1e-3)


@pytest.mark.parametrize("idx", range(5))
def test_launches_of_a_layer_add_up_to_its_algorithmic_bytes(idx):
    """On each schedule a layer's launches carry exactly the per-layer bytes (K
    once, Q_win, the E history read and written, the gather, the indices):
    the K launch and the select launch of a prompt, the one launch of every
    stage on small grids, and the launches of a layer call."""
    wl = inputs.workload(idx)
    kb = lambda n: bench.kernel_bytes(n, wl)
    want = pytest.approx(bench.algorithmic_bytes(wl)["layer_mean"], rel=1e-12)
    select = ("segment_calib", "segment_score", "segment_cand", "final_topk")
    for launches in (("window_score_calib_lse_kr", "segment_select"), ("window_score_single", "segment_select"),
                     ("layer_stages",), ("window_lse_wide", "window_score_calib_wide") + select,
                     ("window_lse_kr", "lse_merge", "window_score_calib_kr") + select):
        assert sum(kb(n) for n in launches) == want


def test_combined_launches_are_sums_of_their_jobs():
    wl = inputs.workload(3)
    kb = lambda n: bench.kernel_bytes(n, wl)
    assert kb("window_score_calib_lse_kr") == pytest.approx(kb("window_score_calib_kr")
                                                          + kb("window_lse_kr"))
    db = lambda n: bench.design_bytes(n, wl)
    assert db("window_score_calib_lse_kr") == pytest.approx(db("window_score_calib_kr")
                                                          + db("window_lse_kr"))
    assert kb("segment_select") == pytest.approx(kb("segment_calib") + kb("segment_score")
                                               + kb("segment_cand") + kb("final_topk"))
    # every stage: both K passes (K read twice) and the select jobs
    assert db("layer_stages") == pytest.approx(db("window_lse_wide") + db("window_score_calib_wide")
                                             + kb("segment_select"))
    K = 32768 * 8 * 128 * 2
    assert db("layer_stages") - kb("layer_stages") == pytest.approx(K + 32 * 32 * 128 * 2 + 32768 * 8 * 4)


@pytest.mark.parametrize("kernel,name", [
    ("void bacon::k_krdual<128, true, 4>(bacon::PassArgs, bacon::PassArgs, bacon::SeqTable)",
     "window_score_calib_lse_kr"),
    ("void bacon::k_pass_dual<true, 128, true>(bacon::PassArgs, bacon::PassArgs, bacon::SeqTable)",
     "window_score_calib_lse"),
    ("void bacon::k_sel<false>(bacon::SegArgs, bacon::SegArgs, bacon::SegArgs, bacon::SegArgs, "
     "bacon::PassArgs, bacon::SeqTable, int, int, int, int, int, bacon::AllocSet<false>)", "segment_select"),
    ("void bacon::k_mega<true, 128, false>(bacon::SegArgs, bacon::SegArgs, bacon::SegArgs, bacon::SegArgs)",
     "layer_stages"),
    ("void bacon::k_wide<0, true, 128>(bacon::PassArgs, bacon::SeqTable)", "window_lse_wide"),
    ("void bacon::k_wide<2, false, 64>(bacon::PassArgs, bacon::SeqTable)", "window_score_calib_wide"),
    ("void bacon::k_sel_one<0>(bacon::SegArgs, bacon::SeqTable)", "segment_score"),
    ("void bacon::k_sel_one<1>(bacon::SegArgs, bacon::SeqTable)", "final_topk"),
    ("void bacon::k_sel_one<2>(bacon::SegArgs, bacon::SeqTable)", "segment_calib"),
    ("void bacon::k_sel_one<3>(bacon::SegArgs, bacon::SeqTable)", "segment_cand"),
    ("void bacon::k_alloc<1>(bacon::AllocArgs, bacon::SeqTable)", "head_alloc"),
    ("bacon::k_split_evidence(bacon::SplitArgs, bacon::SeqTable)", "split_calib"),
])
def test_counter_names(kernel, name):
    assert counters.library_name(kernel) == name


def test_bench_refuses_more_than_one_gpu(monkeypatch, capsys):
    monkeypatch.setattr(sys, "argv", ["bench.py", "--gpus", "2"])
    with pytest.raises(SystemExit) as e:
        bench.main()
    assert e.value.code == 2
    assert "one GPU" in capsys.readouterr().err
