"""Shape bookkeeping against the numbers the paper prints (App. C, Mamba-2 layer FLOP table)."""
import os

from paper_2511_15927_amd import shapes, synth


def golden():
    vals = {}
    for line in open(os.path.join(os.path.dirname(__file__), "golden", "flops_mamba_layer.txt")):
        if line.strip() and not line.startswith("#"):
            k, v = line.split()
            vals[k] = float(v)
    return vals


def test_paper_layer_flops_reproduced():
    g = golden()
    # D_in = 2*d_inner (x, gate) + 2*d_state (B, C, one group) + n_heads (Delta) fixes 120 heads of width 32
    n_heads = int(g["D_in"]) - 2 * int(g["d_inner"]) - 2 * int(g["d_state"])
    assert n_heads == 120 and int(g["d_inner"]) // n_heads == 32
    assert shapes.in_proj_width(3840, 1, 128, n_heads) == g["D_in"]
    assert shapes.conv_channels(3840, 1, 128, 1) == g["conv_ch"]
    f = shapes.paper_flops_per_token(1920, 3840, 128, 4, n_heads)
    # the table prints millions with two decimals (three for the conv), truncated or rounded
    assert abs(f["in_proj"] / 1e6 - g["in_proj_M"]) < 0.01 and f["in_proj"] == 2 * 1920 * 8056
    assert abs(f["conv"] / 1e6 - g["conv_M"]) < 0.001 and f["conv"] == 4096 * 4
    assert abs(f["scan"] / 1e6 - g["scan_M"]) < 0.01 and f["scan"] == 2 * 3840 * 128
    assert abs(f["out_proj"] / 1e6 - g["out_proj_M"]) < 0.01 and f["out_proj"] == 2 * 3840 * 1920
    assert abs(f["one_direction"] / 1e6 - g["one_direction_M"]) < 0.01
    assert abs(f["bidirectional"] / 1e6 - g["bidirectional_M"]) < 0.011   # the table doubles the rounded subtotal


def test_algorithmic_bytes_and_flops_of_the_headline():
    cfg = synth.CONFIGS["headline"]
    tokens = cfg["batch"] * cfg["seqlen"]
    assert shapes.algorithmic_bytes(cfg) == tokens * (3 * 4096 + 2 * 16 + 4096) * 2     # 8 B per token-channel + B, C
    assert shapes.algorithmic_flops(cfg) == tokens * 4096 * (2 * (22 + 7 * 16) + 1)
    assert synth.conv_channels(synth.CONFIGS["paper_1p3b"]) == 4096


def test_stored_counters_count_only_for_kernels_that_exist(tmp_path, monkeypatch):
    """bench.py's stored counters: of a kernel that the library has, summed over the directions' launches of the chunked walk only, and
    nothing from a profile of a kernel that is gone."""
    import bench
    have = sorted(k for k in bench.library_kernels() if "bm::sweep_kernel<16, 2, 0, bm::IoBF16" in k)
    walk = sorted(k for k in bench.library_kernels() if "bm::ssd_wide_kernel<128, 64, 2" in k)
    assert len(have) == 2 and len(walk) >= 4
    (tmp_path / "profiles").mkdir()

    def stored(*sections):
        text = "".join("# kernel: %s\nDURATION_NS_UNDER_PMC=%d\nFETCH_BYTES_PER_LAUNCH=%d\nWRITE_BYTES_PER_LAUNCH=1\n" % s for s in sections)
        (tmp_path / "profiles" / "k_pmc.txt").write_text(text)
        return bench.read_profile("k")

    built = bench.library_kernels()
    monkeypatch.setattr(bench, "library_kernels", lambda: built)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    gone = have[0].replace("<16, 2,", "<16, 2, 0,")
    assert stored((gone, 9, 100)) == ({}, None, None)
    counters, kernel, _ = stored((gone, 9, 100), (have[0], 5, 10), (have[1], 4, 20))
    assert kernel == have[0] and bench.traffic_of(counters) == 11
    counters, kernel, _ = stored((walk[0], 5, 10), (walk[1], 4, 20))
    assert kernel == walk[0] and bench.traffic_of(counters) == 32
    # (a preparation kernel is not the dominant one because the walk has gone)
    prep = next(k for k in built if "bm::ssd_prep_kernel<128, 256>" in k and "stub" not in k)
    assert stored((prep, 1, 10), (walk[0].replace("<128, 64, 2,", "<128, 64, 9,"), 5, 10)) == ({}, None, None)


def test_stored_counters_are_of_kernels_of_the_library():
    """The committed counters that bench.py prints name kernels that are built, the one that takes longest among them."""
    import bench
    for workload, dominant, launches in (("headline", "bm::sweep_kernel<16, 2, 0, bm::IoBF16, 0,", 1), ("headline_m2", "bm::ssd_wide_kernel<128, 64, 2,", 2)):
        counters, kernel, _ = bench.read_profile("sweep_" + workload)
        assert dominant in kernel
        # more than the output alone, which each of a call's launches writes or parks in two bytes
        assert bench.traffic_of(counters) > launches * 2 * 8 * 8192 * 4096
