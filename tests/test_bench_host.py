"""Host-side checks of bench.py: the byte model, the kernel label it prints against the
launch table of the library, and the refusal of more than one GPU."""
import os
import subprocess
import sys

import bench
import paper_2506_15174_amd as spmm

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_algorithmic_bytes_model():
    # int32 row_ptr and col_idx, fp32 values, B read once, C written once
    M, K, nnz, N = 512, 2048, 209715, 128
    assert bench.bytes_min(M, K, nnz, N) == 4 * (M + 1) + 8 * nnz + 4 * K * N + 4 * M * N == 2990492


def test_kernel_label_follows_the_launch_table():
    depth = spmm.load().spmm_chunk_depth
    table = {ufi: tuple(depth(ufi, 8, slices) for slices in (2, 4, 8)) for ufi in (1, 2, 4, 8)}
    for ufi, (d2, d4, d8) in table.items():
        assert bench.kernel_shape(128, ufi) == "S=2,VW=4,D=%d" % d2
        assert bench.kernel_shape(64, ufi) == "S=4,VW=4,D=%d" % d4
        assert bench.kernel_shape(32, ufi) == "S=8,VW=4,D=%d" % d8
        # 128 columns of a 16384-row B exceed one L2, 64 fit: tiles of 64
        assert bench.kernel_shape(128, ufi, 16384).startswith("S=4,VW=4,D=%d" % d4)
        # as two tiles of half the width
        assert bench.kernel_shape(128, ufi, tile_cols=64) == "S=4,VW=4,D=%d, tiles of 64 columns" % d4
        assert bench.kernel_shape(64, ufi, tile_cols=32) == "S=8,VW=4,D=%d, tiles of 32 columns" % d8
        assert bench.kernel_shape(128, ufi, tile_cols=128) == "S=2,VW=4,D=%d" % d2
    # plans made for narrow B: chunks of 16 / 32 / 64 columns on 8 / 16 / 32 or 64 slices, depth by height
    narrow = {ufi: depth(ufi, 16, 8) for ufi in (1, 2, 4, 8)}
    for ufi, d in narrow.items():
        assert bench.kernel_shape(32, ufi, ufk=16) == "S=8,VW=4,D=%d,UFK=16" % d
        assert bench.kernel_shape(16, ufi, ufk=32) == "S=16,VW=4,D=%d,UFK=32" % d
        assert bench.kernel_shape(8, ufi, ufk=64) == "S=32,VW=4,D=%d,UFK=64" % d
        assert bench.kernel_shape(4, ufi, ufk=64) == "S=64,VW=4,D=%d,UFK=64" % d
    assert bench.tiles_of_64(128, 16384) and not bench.tiles_of_64(128, 8192)
    assert not bench.tiles_of_64(64, 16384) and not bench.tiles_of_64(128, 16385)
    # the executor's own condition, as written in its source
    api = open(os.path.join(ROOT, "paper_2506_15174_amd", "csrc", "spmm_api.cpp")).read()
    assert "h.K * 512 > ((int64_t)4 << 20) && (int64_t)h.K * 256 <= ((int64_t)4 << 20)" in api


def test_counter_figures_are_passed_on_only_for_the_profiled_sources(monkeypatch):
    """Traffic and counter figures come from the committed counter summaries, which carry
    the hash of the library sources they were taken on: they are withheld once the sources
    differ, and a plan cut into column ranges is labelled as such."""
    now = bench.kernel_source_hash()
    traffic, prov = bench.measured_traffic("stress", 128)
    assert prov is not None and prov["file"].startswith("profiles/") and prov["source_hash_now"] == now
    assert (traffic is not None) == prov["current"] == (prov["source_hash_at_profile"] == now)
    counters = bench.measured_counters("stress", 128)
    assert (counters is not None) == prov["current"]
    if counters:
        assert set(counters) == {"l2_hit", "valu_busy", "l1_busy"} and all(0 < v <= 100 for v in counters.values())
    monkeypatch.setattr(bench, "kernel_source_hash", lambda: "0" * 16)
    traffic, prov = bench.measured_traffic("stress", 128)
    assert traffic is None and not prov["current"] and prov["withheld_bytes"] > 0
    assert bench.measured_counters("stress", 128) is None
    assert bench.kernel_shape(128, 8, 16384, k_slices=4) == "S=2,VW=4,D=2, 4 column ranges"


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in (r.stdout + r.stderr)


def test_build_refuses_kernel_instances_that_spill():
    """The build parses the compiler's resource remarks and fails when any kernel instance
    uses scratch memory (a spilled register could be an in-flight load destination)."""
    import pytest
    from paper_2506_15174_amd import build
    ok = ("remark: k.hip:1:1: Function Name: kernel_a [-Rpass-analysis=kernel-resource-usage]\n"
          "remark: k.hip:1:1:     VGPRs: 64 [-Rpass-analysis=kernel-resource-usage]\n"
          "remark: k.hip:1:1:     ScratchSize [bytes/lane]: 0 [-Rpass-analysis=kernel-resource-usage]\n"
          "remark: k.hip:1:1:     SGPRs Spill: 0 [-Rpass-analysis=kernel-resource-usage]\n"
          "remark: k.hip:1:1:     VGPRs Spill: 0 [-Rpass-analysis=kernel-resource-usage]\n")
    assert build.check_no_spills(ok) == 1
    with pytest.raises(RuntimeError, match="kernel_a: VGPRs Spill = 3"):
        build.check_no_spills(ok.replace("VGPRs Spill: 0", "VGPRs Spill: 3"))
    with pytest.raises(RuntimeError, match="ScratchSize"):
        build.check_no_spills(ok.replace("lane]: 0", "lane]: 16"))
    with pytest.raises(RuntimeError, match="no resource remarks"):
        build.check_no_spills("")


def test_build_refuses_a_barrier_that_a_load_to_lds_may_cross():
    """The build walks the compiler's assembly back from the barrier behind a strip's copy: the loads that may cross it are the
    entries', on every way."""
    import pytest
    from paper_2506_15174_amd import build
    ok = """
kernel:
        s_cbranch_scc1 .LBB0_2
.LBB0_1:                                ; %copy
        buffer_load_dwordx4 v2, s[0:3], 0 offen lds
        s_cbranch_scc1 .LBB0_1
.LBB0_2:
        buffer_load_dwordx4 v[4:7], v3, s[4:7], 0 offen
        buffer_load_dwordx2 v[8:9], v3, s[4:7], 0 offen
        s_cbranch_vccz .LBB0_4
        s_waitcnt vmcnt(2) lgkmcnt(0)
        s_barrier
.LBB0_4:
        s_endpgm
"""
    entry = "        buffer_load_dwordx2 v[8:9], v3, s[4:7], 0 offen\n"
    copy = "        buffer_load_dwordx4 v2, s[0:3], 0 offen lds\n"
    assert build.check_waits_at_barriers(ok) == 1
    assert build.check_waits_at_barriers(ok.replace("vmcnt(2)", "vmcnt(0)")) == 0  # the compiler's own
    for bad in (ok.replace(entry, ""),                                                      # one load fewer
                ok.replace(entry, copy + entry), ok.replace(entry, entry + copy),           # the copy between them, and after
                ok.replace(entry, entry + "        global_store_dword v1, v2, s[0:1]\n"),   # counted with the loads, in no order with them
                ok.replace(".LBB0_2:", "        s_cbranch_vccz .LBB0_3\n.LBB0_2:").replace(entry, ".LBB0_3:\n" + entry)):  # a way past one of them
        with pytest.raises(RuntimeError, match="all but 2 loads"):
            build.check_waits_at_barriers(bad)
    waited = ok.replace(entry, "        s_waitcnt vmcnt(0)\n" + entry)
    assert build.check_waits_at_barriers(waited) == 1  # one load in flight, and nothing older


def test_facts_of_a_plan_on_tiles():
    """Of a plan on tiles the benchmark prints the tiles' facts and none of the chunk schedule that it does not use."""
    info = spmm.plan_create(3, 4, [0, 2, 2, 3], [0, 3, 1], [1.0, 2.0, 3.0], host_only=True).describe()
    assert bench.schedule_of(info, bench.PLAN_KEYS) == {k: info[k] for k in bench.PLAN_KEYS}
    on_tiles = bench.schedule_of(dict(info, tile_rows=16), bench.PLAN_KEYS)
    assert on_tiles["tile_rows"] == 16 and on_tiles["n_chunks"] == info["n_chunks"]
    assert all(on_tiles[k] is None for k in ("ufi", "group_nnz", "n_blocks", "k_slices", "n_cross"))
    assert bench.tile_kernel(32) == "spmm_tiles_kernel<R=32>" and bench.tile_kernel(8) == "spmm_narrow_tiles_kernel"
    src = open(os.path.join(ROOT, "paper_2506_15174_amd", "csrc", "spmm_tiles.hip")).read()
    assert "void spmm_tiles_kernel(" in src and "void spmm_narrow_tiles_kernel(" in src
