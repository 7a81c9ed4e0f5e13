"""GPU parity of the MLP path: the HIP kernels, called through the C ABI, against the CPU fp64 oracle on
the same seeded inputs, element by element.  Tolerance: max-abs error <= 2e-2 * max|reference| for O, dX and
the three weight gradients (the bar the LM-head gradients are held to; the arithmetic is the same bf16
operand / fp32 accumulate / bf16 intermediate scheme); weight gradients bit-identical across runs."""
import numpy as np
import pytest

import mst_inputs as mi
from oracle import mlp_oracle as orc

pytestmark = pytest.mark.gpu

TOL = 2e-2
NAMES = ("O", "dX", "dWg", "dWu", "dWd")


def _harness():
    from tests.mlp_gpu_harness import MlpDeviceRun, f64
    return MlpDeviceRun, f64


def _reference(inp):
    return orc.mlp(inp.f64("X"), inp.f64("Wg"), inp.f64("Wu"), inp.f64("Wd"), inp.f64("dO"))


def _run_all(inp, M=None, pad=0):
    MlpDeviceRun, f64 = _harness()
    run = MlpDeviceRun(inp, M=M, pad_workspace=pad)
    O = run.forward()
    ws_f = run.last_ws
    dX, dWg, dWu, dWd = run.backward()
    got = {"O": f64(O), "dX": f64(dX), "dWg": f64(dWg), "dWu": f64(dWu), "dWd": f64(dWd)}
    return run, got, ws_f


def _check(inp, M=None):
    ref = _reference(inp)
    run, got, _ = _run_all(inp, M=M)
    errs = {}
    for k in NAMES:
        assert np.isfinite(got[k]).all(), f"{k}: not every element was written"
        scale = max(np.abs(ref[k]).max(), 1e-30)
        errs[k] = float(np.abs(got[k] - ref[k]).max() / scale)
        assert errs[k] <= TOL, f"{k}: max-abs error {errs[k]:.3e} of max|ref|"
    return run, got, ref, errs


def test_tiny_configuration_matches_oracle():
    _, _, _, errs = _check(mi.make_mlp_inputs(1))
    print("mlp cfg1 errors / max|ref|:", {k: f"{v:.2e}" for k, v in errs.items()})


@pytest.mark.parametrize("S,d,I,M", [
    (300, 136, 200, 3),      # nothing a multiple of a tile; last chunk of 100 rows; I % 128 = 72
    (257, 64, 136, 1),       # one row into the second row tile; I % 16 == 8
    (64, 8, 8, 2),           # smallest legal d and I
    (1100, 264, 520, 2),     # several row tiles, several 128-wide and 256-wide tiles of I, ragged everywhere
    (520, 512, 1160, 5),     # d of two tiles; chunks of 104 rows
    (7, 16, 24, 7),          # one row per chunk
])
def test_ragged_shapes_match_oracle(S, d, I, M):
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, M, index=200 + S % 97, w_std=0.05))
    _check(inp)


@pytest.mark.parametrize("S,d,I,M", [
    (57, 656, 1680, 4), (526, 704, 1944, 3), (1920, 320, 584, 1), (513, 144, 1776, 10), (255, 672, 920, 5),
    (1151, 1008, 1184, 4), (2232, 1032, 512, 6), (7, 936, 1984, 5), (1498, 832, 416, 11), (512, 960, 512, 1),
    (257, 704, 1632, 7), (1, 8, 2048, 1),
])
def test_seeded_random_shapes_match_oracle(S, d, I, M):
    """Shapes drawn once from a seeded generator (S around the 255 / 256 / 257 / 512 / 513 tile edges and single rows,
    d from 8 to 1032, I from 416 to 2048, M up to 11, so that d spans several tiles of the dX and weight-gradient
    launches and the chunks are ragged): all five outputs against the oracle."""
    w_std = (0.02, 0.05, 0.3)[(S + I) % 3]
    _check(mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, M, index=300 + (S * 5 + I) % 89, w_std=w_std)))


def test_large_activations_saturate_without_nan():
    # gate pre-activations with |g| up to ~60: exp2 overflows inside the logistic function and must give 0, not NaN
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(256, 128, 256, 2, index=301, x_std=4.0, w_std=0.4))
    _check(inp)


@pytest.mark.parametrize("M", [1, 2, 4, 16])
def test_result_does_not_depend_on_m(M):
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(512, 128, 384, 1, index=302, w_std=0.05))
    _, base, _ = _run_all(inp, M=1)
    _, got, _ = _run_all(inp, M=M)
    # a token's O and dX rows never see the partition: bit-identical
    assert np.array_equal(got["O"], base["O"])
    assert np.array_equal(got["dX"], base["dX"])
    # weight gradients: same terms, different grouping of the fp32 sums
    for k in ("dWg", "dWu", "dWd"):
        scale = np.abs(base[k]).max()
        assert np.abs(got[k] - base[k]).max() <= 1e-5 * scale, k


def test_weight_gradients_are_bit_identical_across_runs():
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(700, 256, 640, 3, index=303, w_std=0.05))
    _, a, _ = _run_all(inp)
    _, b, _ = _run_all(inp)
    for k in NAMES:
        assert np.array_equal(a[k], b[k]), k


def test_zero_upstream_gradient_gives_zero_gradients():
    import torch
    MlpDeviceRun, f64 = _harness()
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(300, 64, 136, 2, index=304))
    run = MlpDeviceRun(inp)
    dX, dWg, dWu, dWd = run.backward(dO=torch.zeros_like(run.dO))
    for t in (dX, dWg, dWu, dWd):
        assert np.abs(f64(t)).max() == 0.0


def test_zero_gate_weights_closed_form():
    # Wg = 0: O = 0, dX = 0, dWu = 0, dWd = 0; dWg = (0.5 * dA * U)^T X  (silu'(0) = 1/2)
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(260, 64, 136, 2, index=305, w_std=0.1))
    inp.Wg_bits[:] = 0
    _, got, ref, _ = _check(inp)
    assert np.abs(got["O"]).max() == 0 and np.abs(got["dX"]).max() == 0
    assert np.abs(got["dWu"]).max() == 0 and np.abs(got["dWd"]).max() == 0
    assert np.abs(ref["dWg"]).max() > 0


def test_workspace_is_respected():
    MlpDeviceRun, _ = _harness()
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(300, 136, 200, 3, index=306))
    run = MlpDeviceRun(inp, pad_workspace=4096)
    run.forward()
    assert (run.last_ws[run.fwd_bytes:].cpu().numpy() == 0xA5).all(), "forward wrote past its declared workspace"
    run.backward()
    assert (run.last_ws[run.bwd_bytes:].cpu().numpy() == 0xA5).all(), "backward wrote past its declared workspace"
    assert run.fwd_bytes == -(-inp.cfg.C * inp.cfg.I * 2 // 256) * 256 or run.fwd_bytes == inp.cfg.C * inp.cfg.I * 2


def test_argument_errors_on_the_device_box():
    import torch
    MlpDeviceRun, _ = _harness()
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(64, 16, 40, 2, index=307))
    run = MlpDeviceRun(inp)
    O = torch.empty((64, 16), dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(run.fwd_bytes, dtype=torch.uint8, device="cuda")
    with pytest.raises(run.mst.MstError) as e:
        run.mst.mst_mlp_fwd(run.X, run.Wg, run.Wu, run.Wd, run.M, ws[: run.fwd_bytes - 256], O)
    assert e.value.status == -4
    with pytest.raises(run.mst.MstError) as e:
        run.mst.mst_mlp_fwd(run.X, run.Wg, run.Wu, run.Wd, 0, ws, O)
    assert e.value.status == -3


def test_repeated_calls_reuse_the_workspace():
    MlpDeviceRun, f64 = _harness()
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(300, 136, 200, 3, index=308))
    ref = _reference(inp)
    run = MlpDeviceRun(inp)
    for _ in range(3):
        O = f64(run.forward())
        assert np.abs(O - ref["O"]).max() <= TOL * np.abs(ref["O"]).max()
        dX = f64(run.backward()[0])
        assert np.abs(dX - ref["dX"]).max() <= TOL * np.abs(ref["dX"]).max()


# (S, d, I, chunkings).  Between them every product takes every tile it can (test_mlp_library_abi.py asks the library which
# ones these are), alone and behind full rounds of large tiles, at ragged edges.
TILE_SHAPES = [
    # ragged in every dimension; between them the launches of the three chunkings take most block tiles: 256 x 256 for
    # gate/up unsplit, 128 x 128, 64 x 64 with the shallow (unsplit) and the deep pipeline (split), last tiles of 4 rows
    (1700, 1160, 4104, (1, 2, 5)),
    # down and dX: 256 x 256 unsplit, 128 x 128 in halves (12 full row tiles, a last column tile of 8); few K steps
    (3000, 4104, 520, (1, 2)),
    # full rounds of large tiles and a second launch with smaller ones behind them: gate/up and dA unsplit
    (1700, 1032, 9800, (1, 2)),
    # the same for down and dX
    (1700, 9480, 1032, (1, 2)),
    # long contractions on few tiles (K steps of 128 in down and dX, the last one ragged), chunks of 65 rows
    (195, 520, 4360, (1, 3)),
    # chunks of 129 rows, forward groups of 257 and 65: one row past a tile of the smaller ones
    (387, 2056, 1032, (3, 6)),
    # down and dX: lone 128 x 128 unsplit; weight gradients of lone 64 x 64 tiles over three chunks
    (7709, 488, 328, (1, 3)),
    # gate/up with K steps of 128, the last one ragged, one and two row tiles
    (61, 4080, 2040, (1, 2)),
    (65, 4104, 1032, (1, 2)),
    # super-tiles of large tiles in down and dX; weight gradients of 64 x 64 tiles in two chunks
    (7995, 1904, 136, (1, 2)),
    # gate/up: super-tiles alone; full rounds, then 128 x 128, 64 x 64, lone 128 x 128
    (3017, 200, 7896, (1, 2)),
    (1982, 272, 10056, (1, 2)),
    (4050, 328, 2512, (1, 2)),
    # the same for dA
    (7954, 152, 1832, (1, 2, 4)),
    (6153, 392, 3200, (1, 2, 4)),
    # the same for down and dX
    (4555, 4352, 264, (1, 2)),
    (7993, 4816, 136, (1, 2)),
    (2612, 7616, 264, (1, 3)),
    (2971, 6616, 360, (1, 2)),
]


@pytest.mark.parametrize("S,d,I,Ms", TILE_SHAPES)
def test_every_block_tile_matches_oracle_and_gives_the_same_bits(S, d, I, Ms):
    """Which block tile a launch takes depends on the rows of a group; a token's O and dX must not.  The weight gradients
    of every chunking (their sums are formed group by group) against the oracle."""
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, Ms[0], index=320 + S % 7, w_std=0.05))
    _, base, ref, _ = _check(inp, M=Ms[0])
    for M in Ms[1:]:
        _, got, _ = _run_all(inp, M=M)
        for k in ("O", "dX"):
            assert np.array_equal(got[k], base[k]), (k, M)
        for k in ("dWg", "dWu", "dWd"):
            assert np.abs(got[k] - ref[k]).max() <= TOL * np.abs(ref[k]).max(), (k, M)


# (S, d, I, {M: how dX of each group of rows is computed}): in a launch of its own, or by that of the weight gradients with 256 x 256
# or 128 x 256 tiles (its own dealt out evenly or in rectangles)
DX_SHAPES = [
    (797, 2080, 1008, {1: ["128"], 2: ["128", "128"], 3: ["64"] * 3}),
    (1661, 1864, 1848, {1: ["own"], 2: ["128", "128"]}),
    (2713, 2264, 808, {1: ["256"], 2: ["128", "256"], 3: ["64"] * 3}),
    (4061, 2000, 1896, {2: ["256", "256"], 3: ["own"] * 3}),
    (673, 5496, 584, {1: ["own"], 2: ["own", "256"]}),        # the tiles of its own launch: 64 x 64 in chunks,
    (2697, 6360, 224, {1: ["own"]}),                         # lone 64 x 64
    (3711, 4392, 312, {1: ["own"]}),                         # and 32 x 32 behind full rounds of large ones
]


@pytest.mark.parametrize("S,d,I,kinds", DX_SHAPES)
def test_dx_beside_the_weight_gradients_matches_oracle_and_keeps_its_bits(S, d, I, kinds):
    MlpDeviceRun, _ = _harness()
    import paper_2407_15892_amd as mst
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, 1, index=330 + S % 7, w_std=0.05))
    base = None
    for M, want in kinds.items():
        assert [g["dx"] for g in mst.mst_mlp_bwd_groups(S, d, I, M)] == want
        _, got, _, _ = _check(inp, M=M)
        base = got["dX"] if base is None else base
        assert np.array_equal(got["dX"], base), M      # a token's dX does not depend on who computed it


@pytest.mark.parametrize("S,d,I,kinds", [
    (833, 1544, 4616, {1: [128], 2: [0, 128]}),          # ragged everywhere: a last row tile of 65 and of 32 rows
    (1929, 1032, 2584, {1: [256], 2: [128, 128]}),       # first chunk in tiles of 256 rows, of 965 in 128 x 128; one row, 8 columns
    (385, 2184, 5464, {1: [128]}),                       # one row past three row tiles, last K steps ragged
])
def test_dx_in_128_by_128_tiles_beside_the_weight_gradients(S, d, I, kinds):
    import paper_2407_15892_amd as mst
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, 1, index=370 + S % 7, w_std=0.05))
    base = None
    for M, want in list(kinds.items()) + [(max(2, S // 60), None)]:      # the last in groups of up to 140 rows, launches of their own
        got_rows = [g["dx_tile_rows"] for g in mst.mst_mlp_bwd_groups(S, d, I, M)]
        assert got_rows == want if want else 128 not in got_rows, (M, got_rows)
        _, got, _, _ = _check(inp, M=M)
        base = got["dX"] if base is None else base
        assert np.array_equal(got["dX"], base), M


# (S, d, I, {M: (how dX of every group of rows is computed, dA in the launch of gate/up's backward)}): the launches of small problems,
# and 32 x 32 tiles in every product that takes them
SMALL_SHAPES = [
    (65, 264, 904, {1: ("32", True), 2: ("32", True)}),       # last tiles of one row, of 8 columns
    (513, 264, 776, {1: ("32", True), 5: ("32", True)}),
    (1, 8, 8, {1: ("32", True)}),                             # fewer K than one step
    (97, 72, 40, {3: ("32", True)}),
    (33, 1032, 2056, {1: ("32", False), 2: ("32", False)}),   # dA in 32 x 32 tiles
    (450, 776, 1992, {1: ("64", True), 7: ("32", True)}),
    (2001, 264, 1032, {1: ("64", False), 2: ("64", False)}),
    (5083, 472, 368, {1: ("64", False), 2: ("64", True)}),    # unsplit: the weight gradients' longer tiles before 640 of dX
    (41, 2056, 4104, {1: ("own", False)}),                    # dX in 32 x 32 tiles, its last K step of 128 ragged
    (300, 520, 16, {1: ("32", True)}),
]


@pytest.mark.parametrize("S,d,I,kinds", SMALL_SHAPES)
def test_launches_of_small_problems_match_oracle_and_keep_their_bits(S, d, I, kinds):
    MlpDeviceRun, _ = _harness()
    import paper_2407_15892_amd as mst
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, 1, index=340 + S % 7, w_std=0.05))
    base = None
    for M, (dx, da) in kinds.items():
        groups = mst.mst_mlp_bwd_groups(S, d, I, M)
        assert {g["dx"] for g in groups} == {dx} and {g["da_in_gateup"] for g in groups} == {da}
        _, got, _, _ = _check(inp, M=M)
        base = got if base is None else base
        for k in ("O", "dX"):
            assert np.array_equal(got[k], base[k]), (k, M)
    # the same tokens behind rows that give the chunk large tiles
    C = 1024
    wide = mi.make_mlp_inputs(mi.custom_mlp_config(S + C, d, I, 1, index=341, w_std=0.05))
    for name in ("Wg", "Wu", "Wd"):
        getattr(wide, name + "_bits")[:] = getattr(inp, name + "_bits")
    for name in ("X", "dO"):
        getattr(wide, name + "_bits")[C:] = getattr(inp, name + "_bits")
    _, got, _ = _run_all(wide, M=1)
    for k in ("O", "dX"):
        assert np.array_equal(got[k][C:], base[k]), k


@pytest.mark.parametrize("S,d,I,products,M", [
    (1281, 4104, 2056, ("gateup", "down"), 3),    # last tiles of one row, of 8 indices and columns
    (700, 1032, 4104, ("gateup",), 2),
    (1486, 264, 8008, ("gateup",), 2),            # behind a round of large ones
    (4402, 4744, 1256, ("down",), 7),
])
def test_tiles_of_128_by_256_match_oracle_and_keep_their_bits(S, d, I, products, M):
    import paper_2407_15892_amd as mst
    whole = mst.mst_mlp_tile_info(S, d, I)
    for rows, _ in mst.mst_mlp_fwd_groups(S, d, I, M):
        assert all(whole[p][0] == "128x256" != mst.mst_mlp_tile_info(rows, d, I)[p][0] for p in products)
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, 1, index=350 + S % 7, w_std=0.05))
    _, base, _, _ = _check(inp, M=1)
    _, got, _ = _run_all(inp, M=M)
    for k in ("O", "dX"):
        assert np.array_equal(got[k], base[k]), k


@pytest.mark.parametrize("S,d,I,M", [
    (1500, 136, 264, 12),     # chunks of 125 rows; several groups of rows with their A in the output, the last ones in the workspace
    (1601, 264, 520, 23),     # ragged everywhere, groups of odd numbers of rows
    (700, 520, 72, 9),        # I < d: the output holds most of A at once
    (131, 8, 1032, 4),        # I much larger than d: nothing of it
])
def test_forward_groups_of_rows_keep_the_bits(S, d, I, M):
    """Where the forward keeps A -- in the declared workspace, in a larger one, in rows of O that are not written yet -- does
    not show in O, and it stays inside both.  An O that is X itself (its rows are read before they are written, chunk by
    chunk) holds no A."""
    import torch
    MlpDeviceRun, f64 = _harness()
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, M, index=360 + S % 7, w_std=0.05))
    run = MlpDeviceRun(inp, M=M)
    ref = _reference(inp)["O"]
    base = f64(MlpDeviceRun(inp, M=1).forward())
    assert np.abs(base - ref).max() <= TOL * np.abs(ref).max()
    for times in (1, 2, 3):
        ws = torch.full((times * run.fwd_bytes + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        O = torch.full(((S + 2) * d,), float("nan"), dtype=torch.bfloat16, device="cuda")
        run.mst.mst_mlp_fwd(run.X, run.Wg, run.Wu, run.Wd, M, ws[: times * run.fwd_bytes], O[d:-d].view(S, d))
        torch.cuda.synchronize()
        assert np.array_equal(f64(O[d:-d].view(S, d)), base), times
        assert bool((ws[times * run.fwd_bytes:] == 0xA5).all()) and bool(O[:d].isnan().all()) and bool(O[-d:].isnan().all())
    X = run.X.clone()
    run.mst.mst_mlp_fwd(X, run.Wg, run.Wu, run.Wd, M, ws[: run.fwd_bytes], X)
    torch.cuda.synchronize()
    assert np.array_equal(f64(X), base)


@pytest.mark.parametrize("S,d,I,M", [
    (1500, 136, 264, 12),     # one or two of dG, dU and A in dX behind the group, the last groups' all in the workspace
    (1601, 264, 520, 23),     # ragged everywhere
    (2401, 72, 168, 80),      # all three of them first
    (5207, 520, 1304, 11),    # larger tiles
    (700, 520, 72, 9),        # I < d
    (131, 8, 1032, 4),        # I much larger than d: nothing in dX
])
def test_backward_groups_of_rows_match_oracle_and_keep_the_bits_of_dx(S, d, I, M):
    """Where the backward keeps dG, dU and A does not show in dX, and it stays inside the declared workspace and dX."""
    import torch
    MlpDeviceRun, f64 = _harness()
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, M, index=380 + S % 7, w_std=0.05))
    ref = _reference(inp)
    base = f64(MlpDeviceRun(inp, M=1).backward()[0])
    assert np.abs(base - ref["dX"]).max() <= TOL * np.abs(ref["dX"]).max()
    run = MlpDeviceRun(inp, M=M)
    for times in (1, 2):
        ws = torch.full((times * run.bwd_bytes + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
        dX = torch.full(((S + 2) * d,), float("nan"), dtype=torch.bfloat16, device="cuda")
        dW = [torch.full(shape, float("nan"), device="cuda") for shape in ((I, d), (I, d), (d, I))]
        run.mst.mst_mlp_bwd(run.X, run.Wg, run.Wu, run.Wd, run.dO, M, ws[: times * run.bwd_bytes], dX[d:-d].view(S, d), *dW)
        torch.cuda.synchronize()
        assert np.array_equal(f64(dX[d:-d].view(S, d)), base), times
        for k, got in zip(("dWg", "dWu", "dWd"), dW):
            assert np.abs(got.double().cpu().numpy() - ref[k]).max() <= TOL * np.abs(ref[k]).max(), (k, times)
        assert bool((ws[times * run.bwd_bytes:] == 0xA5).all()) and bool(dX[:d].isnan().all()) and bool(dX[-d:].isnan().all())


@pytest.mark.parametrize("S,d,I,M", [
    (1500, 136, 264, 12),
    (1601, 264, 520, 23),
    (2612, 776, 264, 3),      # chunk by chunk
    (300, 72, 8, 37),         # chunks of nine rows, whose 144 bytes a buffer are rounded up to 256
])
def test_weight_gradients_keep_their_bits_in_a_larger_workspace(S, d, I, M):
    """The order of their sums depends on the shape alone, and of a larger workspace nothing but the declared size is written."""
    import torch
    MlpDeviceRun, _ = _harness()
    run = MlpDeviceRun(mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, M, index=385, w_std=0.05)))
    base = run.backward()
    for more in (256, run.bwd_bytes, 7 * run.bwd_bytes):
        run.pad = more
        ws = run._ws(run.bwd_bytes)
        got = [torch.full_like(t, float("nan")) for t in base]
        run.mst.mst_mlp_bwd(run.X, run.Wg, run.Wu, run.Wd, run.dO, M, ws, *got)
        torch.cuda.synchronize()
        for a, b in zip(got, base):
            assert torch.equal(a.view(torch.int16 if a.dtype == torch.bfloat16 else torch.int32),
                               b.view(torch.int16 if a.dtype == torch.bfloat16 else torch.int32)), more
        assert bool((ws[run.bwd_bytes:] == 0xA5).all()), more


@pytest.mark.parametrize("of", ["X", "dO"])
def test_dx_that_overlaps_rows_already_read_is_formed_chunk_by_chunk(of):
    """dX a chunk of rows before X or dO in the same buffer: a chunk's rows are overwritten after they have been read.  Without
    the overlap this shape takes fewer, larger groups of rows."""
    import torch
    MlpDeviceRun, f64 = _harness()
    S, d, I, M = 1500, 136, 264, 12
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, M, index=386, w_std=0.05))
    ref = _reference(inp)
    run = MlpDeviceRun(inp)
    base = run.backward()
    C = S // M
    both = torch.empty((S + C, d), dtype=torch.bfloat16, device="cuda")
    both[C:] = getattr(run, of)
    ins = {"X": run.X, "dO": run.dO, of: both[C:]}
    got = [both[:S]] + [torch.full_like(t, float("nan")) for t in base[1:]]
    ws = run._ws(run.bwd_bytes)
    run.mst.mst_mlp_bwd(ins["X"], run.Wg, run.Wu, run.Wd, ins["dO"], M, ws, *got)
    torch.cuda.synchronize()
    assert torch.equal(got[0].view(torch.int16), base[0].view(torch.int16))
    for k, t in zip(NAMES[2:], got[1:]):
        assert np.abs(f64(t) - ref[k]).max() <= TOL * np.abs(ref[k]).max(), k


@pytest.mark.parametrize("S,d,I,M", [
    (1537, 712, 2312, 4),      # rows of 4624 bytes, 16 behind a line one after the other; a last K step of 8, last tiles of one row
    (2049, 520, 2072, 3),      # odd multiples of 8
    (1990, 584, 2136, 5),      # rows of 4272 bytes: 48 behind
    (1100, 1160, 4104, 6),     # the last K step's chunks reach into one more stage for some rows only
])
def test_down_of_rows_that_are_not_whole_lines_keeps_its_bits(S, d, I, M):
    """Down in lone 64 x 64 tiles, more of them than compute units: the same bits as chunk by chunk, where fewer tiles load the
    same k of all rows."""
    import torch
    import paper_2407_15892_amd as mst
    MlpDeviceRun, f64 = _harness()
    assert "down" in mst.mst_mlp_line_panels(S, d, I)
    assert all("down" not in mst.mst_mlp_line_panels(rows, d, I) for rows, _ in mst.mst_mlp_fwd_groups(S, d, I, M))
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, M, index=390 + S % 7, w_std=0.05))
    run = MlpDeviceRun(inp, M=1)
    whole = f64(run.forward())
    assert np.abs(whole - _reference(inp)["O"]).max() <= TOL * np.abs(_reference(inp)["O"]).max()
    assert np.array_equal(f64(MlpDeviceRun(inp, M=M).forward()), whole)
    C = -(-S // M)
    O = torch.empty((C, d), dtype=torch.bfloat16, device="cuda")          # every chunk as a call of its own
    ws = torch.empty(run.fwd_bytes, dtype=torch.uint8, device="cuda")
    for r0 in range(0, S, C):
        n = min(C, S - r0)
        mst.mst_mlp_fwd(run.X[r0:r0 + n], run.Wg, run.Wu, run.Wd, 1, ws, O[:n])
        torch.cuda.synchronize()
        assert np.array_equal(f64(O[:n]), whole[r0:r0 + n]), r0


def _offset(t, elements):
    """A copy of t that begins `elements` elements behind a line."""
    import torch
    buf = torch.empty(t.numel() + 64 + elements, dtype=t.dtype, device="cuda")
    first = -buf.data_ptr() // t.element_size() % (128 // t.element_size()) + elements
    out = buf[first:first + t.numel()].view(t.shape)
    out.copy_(t)
    return out


@pytest.mark.parametrize("S,d,I,M,elements", [
    (3023, 584, 496, 19, 0),       # the first groups' A in rows of O, 48 bytes behind a line
    (1537, 712, 2312, 1, 8),       # weights 16 bytes behind a line, A on one
    (1152, 1024, 1088, 1, 56),     # rows that are whole lines, all beginning 112 bytes behind one
])
def test_down_by_lines_wherever_its_operands_begin(S, d, I, M, elements):
    """Line panels of operands that do not begin on a line: the same bits as where they do, or as where fewer tiles load the
    same k of all rows."""
    import torch
    import paper_2407_15892_amd as mst
    MlpDeviceRun, f64 = _harness()
    if M > 1:
        rows, in_output = mst.mst_mlp_fwd_groups(S, d, I, M)[0]
        assert in_output and 2 * (S * d - rows * I) % 128 == 48 and "down" in mst.mst_mlp_line_panels(rows, d, I)
    else:
        assert mst.mst_mlp_tile_info(S, d, I)["down"][:2] == ("64_lone", 0) and -(-S // 64) * -(-d // 64) > 256
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, M, index=400 + S % 7, w_std=0.05))
    run = MlpDeviceRun(inp)
    ref = _reference(inp)["O"]
    O = _offset(torch.full((S, d), float("nan"), dtype=torch.bfloat16, device="cuda"), 0)
    ws = run._ws(run.fwd_bytes)
    run.mst.mst_mlp_fwd(run.X, run.Wg, run.Wu, _offset(run.Wd, elements), M, ws, O)
    torch.cuda.synchronize()
    got = f64(O)
    assert np.abs(got - ref).max() <= TOL * np.abs(ref).max()
    part = torch.empty((500, d), dtype=torch.bfloat16, device="cuda")
    assert "down" not in mst.mst_mlp_line_panels(500, d, I)
    ws = torch.empty(mst.mst_mlp_workspace_bytes(500, d, I, 1)[0], dtype=torch.uint8, device="cuda")
    for r0 in range(0, S, 500):
        n = min(500, S - r0)
        mst.mst_mlp_fwd(run.X[r0:r0 + n], run.Wg, run.Wu, run.Wd, 1, ws, part[:n])
        torch.cuda.synchronize()
        assert np.array_equal(f64(part[:n]), got[r0:r0 + n]), r0


@pytest.mark.parametrize("S,d,I,product,dx", [
    (515, 264, 1808, "da", "32"),          # rows of dO of 528 bytes; a last row tile of three
    (648, 1512, 1384, "dx", "own"),        # both terms, each with a stage behind its last; rows of 2768 bytes
    (793, 1336, 3368, "dx", "own"),
    (668, 400, 520, "dx", "64"),           # beside the weight gradients
])
def test_gradients_by_lines_keep_their_bits(S, d, I, product, dx):
    """dA and dX in lone 64 x 64 tiles whose token rows are loaded line by line: dX has the bits of the same rows in calls that
    are too short for that."""
    import torch
    import paper_2407_15892_amd as mst
    MlpDeviceRun, f64 = _harness()
    assert product in mst.mst_mlp_line_panels(S, d, I) and mst.mst_mlp_dx_tile(S, d, I, True) == dx
    inp = mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, 1, index=410 + S % 7, w_std=0.05))
    run, got, _, _ = _check(inp)
    ws = torch.empty(mst.mst_mlp_workspace_bytes(100, d, I, 1)[1], dtype=torch.uint8, device="cuda")
    dX = torch.empty((100, d), dtype=torch.bfloat16, device="cuda")
    dW = [torch.empty(shape, device="cuda") for shape in ((I, d), (I, d), (d, I))]
    assert product not in mst.mst_mlp_line_panels(100, d, I)
    for r0 in range(0, S, 100):
        n = min(100, S - r0)
        mst.mst_mlp_bwd(run.X[r0:r0 + n], run.Wg, run.Wu, run.Wd, run.dO[r0:r0 + n], 1, ws, dX[:n], *dW)
        torch.cuda.synchronize()
        assert np.array_equal(f64(dX[:n]), got["dX"][r0:r0 + n]), r0


@pytest.mark.parametrize("S,d,I,M", [
    (1500, 136, 264, 12),      # A in O, one or two of dG, dU and A in dX, small tiles
    (1929, 1032, 2584, 2),     # dX in 128 x 128 tiles
    (3023, 584, 496, 19),      # rows of A line by line
])
def test_forward_and_backward_replay_from_a_hip_graph(S, d, I, M):
    """Nothing but kernels is enqueued: every replay, with eager work and synchronisation in between, gives the eager bits,
    also where intermediates are kept in rows of O and dX."""
    import torch
    MlpDeviceRun, _ = _harness()
    run = MlpDeviceRun(mi.make_mlp_inputs(mi.custom_mlp_config(S, d, I, M, index=420 + S % 7, w_std=0.05)))
    eager = [run.forward().clone()] + [t.clone() for t in run.backward()]
    out = [torch.empty_like(t) for t in eager]
    ws = run._ws(run.bwd_bytes)

    def step():
        run.mst.mst_mlp_fwd(run.X, run.Wg, run.Wu, run.Wd, M, ws, out[0])
        run.mst.mst_mlp_bwd(run.X, run.Wg, run.Wu, run.Wd, run.dO, M, ws, *out[1:])

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for _ in range(3):
        for t in out:
            t.fill_(float("nan"))
        ws.fill_(0xA5)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, eager):
            bits = torch.int16 if a.dtype == torch.bfloat16 else torch.int32
            assert torch.equal(a.view(bits), b.view(bits))
    del graph
