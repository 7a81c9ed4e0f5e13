"""CPU checks of bench.py's host-side helpers (no GPU; of the library only host queries)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_traffic_table_parses_and_covers_the_default_workloads():
    sys.path.insert(0, ROOT)
    import bench
    for kernel in ("fwd_gemm_lse", "bwd_gemm_dlogits", "bwd_gemm_dh", "bwd_gemm_dw"):
        for config in (2, 3):
            t = bench.pmc_traffic_bytes("lmhead", config, "blocks", kernel)
            assert t is not None and 1e9 < t < 1e11, (config, kernel, t)
    # per 1024 rows the forward launch fetches what one mini-sequence's launch used to: about 1.6 GB
    assert 1.5e9 < bench.pmc_traffic_bytes("lmhead", 3, "blocks", "fwd_gemm_lse") / 32 < 1.8e9
    assert bench.pmc_traffic_bytes("mlp", 2, "anything", "dw") > 3e9          # schedule column "-" matches any
    assert bench.pmc_traffic_bytes("lmhead", 4, "blocks", "bwd_gemm_dw") is None
    assert bench.pmc_traffic_bytes("lmhead", 3, "pairs", "bwd_gemm_dw") is None


def test_flop_of_products_that_share_a_launch_are_counted_where_they_run():
    import bench
    apart = {"gateup": 6, "down": 6, "da": 6, "gateup_bwd": 6, "dx": 6, "dw": 6}
    assert bench.mlp_flop_units(apart) == bench.MLP_FLOP_UNITS
    # the small forms: dA inside gate/up's backward, dX beside the weight gradients
    joint = bench.mlp_flop_units(dict(apart, da=0, dx=0))
    assert joint == dict(bench.MLP_FLOP_UNITS, da=0.0, gateup_bwd=6.0, dx=0.0, dw=10.0)
    # a step's first of three chunks with a dX launch of its own, the later ones without
    mixed = bench.mlp_flop_units(dict(apart, dx=2))
    assert abs(mixed["dx"] - 4 / 3) < 1e-12 and abs(mixed["dw"] - (6 + 8 / 3)) < 1e-12
    for units in (joint, mixed):
        assert abs(sum(units.values()) - 22.0) < 1e-12


def test_flop_of_groups_of_rows_are_counted_by_their_rows():
    import bench
    import paper_2407_15892_amd as mst
    groups = mst.mst_mlp_bwd_groups(32768, 4096, 14336, 8)
    assert len({g["rows"] for g in groups}) > 1 and {g["dx"] == "own" for g in groups} == {True, False}
    issued = {"gateup": 8, "down": 8, "da": len(groups), "gateup_bwd": len(groups), "dx": sum(g["dx"] == "own" for g in groups), "dw": len(groups)}
    units = bench.mlp_flop_units(issued, groups)
    own = sum(g["rows"] for g in groups if g["dx"] == "own") / 32768
    assert abs(units["dx"] - 4 * own) < 1e-12 and abs(units["dw"] - (6 + 4 * (1 - own))) < 1e-12 and units["da"] == 2.0
    assert abs(sum(units.values()) - 22.0) < 1e-12


def test_the_order_that_runs_is_named_and_its_flop_counted():
    import bench
    import mst_inputs as mi
    import paper_2407_15892_amd as mst
    cfg = mi.CONFIGS[1]
    shape = (cfg.S, cfg.d, cfg.V, cfg.M)
    assert bench.backward_schedule(mst, *shape) == {"schedule": "streamed", "form": "256_split", "dh_split": 4}
    assert bench.backward_schedule(mst, *shape, "pairs")["schedule"] == "pairs"
    assert bench.backward_schedule(mst, 32768, 4096, 128256, 32)["schedule"] == "blocks_fused"
    # forward 2; the one launch of the streamed backward: logits twice, dH, dW
    assert bench.gemm_kinds("streamed") == dict(bench.GEMM_KINDS, bwd_gemm_dlogits=8.0)
    for schedule in ("pairs", "blocks", "blocks_fused"):
        assert bench.gemm_kinds(schedule) == bench.GEMM_KINDS


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True)
    assert r.returncode == 2 and "ONE GPU" in r.stderr
