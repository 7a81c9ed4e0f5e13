"""CPU-side checks of the MLP C-ABI library: it loads, exports every symbol its header declares, and its
host-only logic (workspace sizing, chunk policy, argument validation) behaves.  No kernel is launched here."""
import os
import re

import pytest

import mst_inputs as mi

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def mst():
    import paper_2407_15892_amd as m
    if not os.path.exists(m.mlp_binding.MLP_LIB_PATH) or not os.path.exists(m.binding.LIB_PATH):
        from paper_2407_15892_amd.build import build
        build()
    m.load_mlp_library()
    return m


def test_every_declared_symbol_is_exported(mst):
    text = open(os.path.join(ROOT, "include", "mst_mlp.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = set(re.findall(r"\b(mst_mlp_[a-z_]+)\s*\(", text))
    assert {"mst_mlp_fwd", "mst_mlp_bwd", "mst_mlp_workspace_bytes", "mst_mlp_suggest_m"} <= names
    lib = mst.load_mlp_library()
    for n in sorted(names):
        assert hasattr(lib, n), f"{n} is declared in the header but not exported"
    assert "gfx950" in mst.mst_mlp_version()
    kinds = [lib.mst_mlp_profile_kind_name(i).decode() for i in range(mst.mlp_binding.MLP_PROFILE_KINDS)]
    assert kinds == ["gateup", "down", "da", "gateup_bwd", "dx", "dw"]
    assert lib.mst_mlp_profile_kind_name(mst.mlp_binding.MLP_PROFILE_KINDS).decode() == "?"


def test_workspace_is_chunk_sized(mst):
    for cfg in mi.MLP_CONFIGS.values():
        f, b = mst.mst_mlp_workspace_bytes(cfg.S, cfg.d, cfg.I, cfg.M)
        assert f == cfg.C * cfg.I * 2, cfg.name          # one chunk of the bf16 intermediate
        assert b == 3 * f, cfg.name                      # dA/dG, dU, A
        # the standard block would hold S x I; the chunked one holds 1/M of it
        assert f * cfg.M == cfg.S * cfg.I * 2
    _, b1 = mst.mst_mlp_workspace_bytes(8192, 4096, 14336, 2)
    _, b2 = mst.mst_mlp_workspace_bytes(32768, 4096, 14336, 8)    # same chunk, 4x the sequence
    assert b1 == b2


def test_chunk_policy_constant_chunk_equal_to_hidden_size(mst):
    sm = mst.mst_mlp_suggest_m
    assert sm(8192, 4096, 14336) == 2
    assert sm(32768, 4096, 14336) == 8
    assert sm(16384, 4096, 11008) == 4
    assert sm(1024, 4096, 14336) == 1      # sequence shorter than the chunk: no split
    assert sm(4096, 4096, 14336) == 1
    assert sm(10000, 4096, 14336) == 2     # nearest integer
    assert sm(0, 4096, 14336) == 0 and sm(8, 0, 8) == 0
    for cfg in mi.MLP_CONFIGS.values():
        assert sm(cfg.S, cfg.d, cfg.I) == cfg.M, cfg.name


def test_shape_and_m_validation(mst):
    st = mst.mlp_binding.mst_mlp_workspace_bytes_status
    assert st(8, 16, 32, 1) == 0
    assert st(0, 16, 32, 1) == -2
    assert st(8, 0, 32, 1) == -2
    assert st(8, 16, 0, 1) == -2
    assert st(8, 12, 32, 1) == -2            # d % 8 != 0
    assert st(8, 16, 36, 1) == -2            # I % 8 != 0
    assert st(8, 16, 32, 0) == -3
    assert st(8, 16, 32, 9) == -3            # M > S
    assert st(8, 1 << 16, 1 << 16, 1) == -2  # I * d >= 2^31
    assert st(1 << 20, 8, 1 << 15, 1) == -2  # one chunk of the intermediate >= 2^30 elements


def test_null_workspace_and_alignment_errors_come_before_any_launch(mst):
    lib = mst.load_mlp_library()
    S, d, I, M = 64, 16, 40, 2
    f, b = mst.mst_mlp_workspace_bytes(S, d, I, M)
    fake = 0x1000    # never dereferenced: validation fails first
    assert lib.mst_mlp_fwd(None, fake, fake, fake, S, d, I, M, fake, f, fake, None) == -1
    assert lib.mst_mlp_fwd(fake, fake, fake, fake, S, d, I, M, fake, f, None, None) == -1
    assert lib.mst_mlp_fwd(fake, fake, fake, fake, S, d, I, M, fake, f - 1, fake, None) == -4
    assert lib.mst_mlp_fwd(fake, fake, fake, fake, S, d, I, M, None, f, fake, None) == -4
    assert lib.mst_mlp_fwd(fake + 8, fake, fake, fake, S, d, I, M, fake, f, fake, None) == -5
    assert lib.mst_mlp_fwd(fake, fake, fake, fake, S, d, I, M, fake + 16, f, fake, None) == -5
    assert lib.mst_mlp_bwd(fake, fake, fake, fake, None, S, d, I, M, fake, b, fake, fake, fake, fake, None) == -1
    assert lib.mst_mlp_bwd(fake, fake, fake, fake, fake, S, d, I, M, fake, b, fake, fake, fake, None, None) == -1
    assert lib.mst_mlp_bwd(fake, fake, fake, fake, fake, S, d, I, M, fake, b - 1, fake, fake, fake, fake, None) == -4
    assert lib.mst_mlp_bwd(fake, fake, fake, fake, fake, S, d, I, M, fake, b, fake, fake + 2, fake, fake, None) == -5
    assert lib.mst_mlp_bwd(fake, fake, fake, fake, fake, S, d, I, 0, fake, b, fake, fake, fake, fake, None) == -3


def test_tile_shapes_of_the_gpu_test_take_every_tile(mst):
    """The library's own answer to which block tiles the shapes of the GPU tests run with, group of rows by group of rows:
    every tile of every product alone, large tiles in both maps, every smaller tile (the rare one with K steps of 128 aside)
    behind full rounds of large ones, and every tile of the weight gradients in a first and in a later group."""
    from tests.test_gpu_mlp_parity import DX_SHAPES, TILE_SHAPES
    seen = set()
    for S, d, I, Ms in TILE_SHAPES + [(S, d, I, tuple(kinds)) for S, d, I, kinds in DX_SHAPES]:
        for M in Ms:
            forward, backward = mst.mst_mlp_fwd_groups(S, d, I, M), mst.mst_mlp_bwd_groups(S, d, I, M)
            launches = [(product, rows) for rows, _ in forward for product in ("gateup", "down")]
            for g in backward:
                launches += [("gateup", g["rows"])] + [("da", g["rows"])] * (not g["da_in_gateup"]) + [("dx", g["rows"])] * (g["dx"] == "own")
            for product, rows in launches:
                tile, head, super_tiles = mst.mst_mlp_tile_info(rows, d, I)[product]
                assert 0 <= head < (I if product in ("gateup", "da") else d) and (head == 0 or tile != "256")
                seen.add((product, tile, super_tiles if tile == "256" else head > 0))
            tile, even = mst.mst_mlp_tile_info(max(g["rows"] for g in backward), d, I)["dw"]
            assert {g["dw"] for g in backward} == {tile}
            seen |= {("dw", tile, even, min(i, 1)) for i in range(len(backward))}
    want = {("dw", t, e, c) for t, e in (("256", False), ("256", True), ("64", True), ("64_lone", True)) for c in (0, 1)}
    for product in ("gateup", "down", "da", "dx"):
        want |= {(product, "256", False), (product, "256", True), (product, "64_long", False)}
        want |= {(product, t, tail) for t in ("128", "128_lone", "64", "64_lone") for tail in (False, True)}
    assert want <= seen, sorted(want - seen)


def test_groups_of_rows_fit_the_memory_they_are_kept_in(mst):
    """Over random shapes: the groups make up the rows, what they keep fits into the workspace and into the rows behind them,
    there are no more of them than chunks, and those of the backward are the chunks where dX is not free."""
    import random
    rng = random.Random(20240718)
    seen = set()
    for _ in range(4000):
        S, d, I = round(2 ** rng.uniform(0, 14)), 8 * round(2 ** rng.uniform(0, 9)), 8 * round(2 ** rng.uniform(0, 10))
        M = rng.randint(1, min(S, 80))
        C = -(-S // M)
        chunks = [min(C, S - r) for r in range(0, S, C)]
        need, need_bwd = mst.mst_mlp_workspace_bytes(S, d, I, M)
        for workspace, overlaps in ((need, False), (need, True), (need_bwd, False), (need + 256 * rng.randint(0, 2000), False)):
            left = S
            groups = mst.mst_mlp_fwd_groups(S, d, I, M, workspace, overlaps)
            for rows, in_output in groups:
                left -= rows
                assert rows > 0 and rows * I < 2 ** 30 and rows * d < 2 ** 30
                assert rows * I <= left * d if in_output else rows * I * 2 <= workspace
                assert not (in_output and overlaps)
                seen.add(("A", in_output))
            assert left == 0 and len(groups) <= len(chunks)
        left = S
        groups = mst.mst_mlp_bwd_groups(S, d, I, M)
        for g in groups:
            rows, k = g["rows"], g["in_dx"]
            left -= rows
            assert rows > 0 and rows * I < 2 ** 30 and rows * d < 2 ** 30 and k * rows * I <= left * d
            assert k == 3 or rows * I * 2 <= need_bwd // (3 - k) // 256 * 256
            seen.add(("dX", k))
        assert left == 0 and len(groups) <= len(chunks)
        assert [g["rows"] for g in mst.mst_mlp_bwd_groups(S, d, I, M, dx_overlaps=True)] == chunks
    assert seen == {("A", False), ("A", True)} | {("dX", k) for k in range(4)}
    lib = mst.load_mlp_library()
    assert lib.mst_mlp_fwd_groups(64, 16, 40, 2, 256, 0, 0, None) == -1      # less than one chunk of A
    assert lib.mst_mlp_fwd_groups(64, 16, 40, 2, 1 << 20, 0, 1, None) == -1
    assert lib.mst_mlp_bwd_groups(64, 16, 40, 65, 0, 0, None) == -1
    assert lib.mst_mlp_line_panels(64, 12, 40) == -1


def test_down_of_65_to_96_tokens_takes_32_by_32_tiles_only_for_short_contractions(mst):
    """Three rows of them, more than one round and a long contraction: 64 x 64 tiles are faster."""
    down = lambda rows, d, I: mst.mst_mlp_tile_info(rows, d, I)["down"][0]
    for rows in (33, 64, 97, 128):
        assert down(rows, 4096, 14336) == "32"
    for rows in (65, 80, 96):
        assert down(rows, 4096, 14336) == "64_long"       # 384 tiles, 224 K steps
        assert down(rows, 3200, 12736) == "32"            # 300 tiles, 199 K steps
        assert down(rows, 3200, 12800) == "64_long"       # 300 tiles, 200 K steps
        assert down(rows, 2720, 16384) == "32"            # one round


def test_down_takes_line_panels_in_place_of_128_by_128_tiles_only_where_they_are_faster(mst):
    """A few more 128 x 128 tiles than compute units, and rows that begin anywhere in a line."""
    down = lambda rows, d, I: mst.mst_mlp_tile_info(rows, d, I)["down"][:2]
    assert down(1169, 3296, 11048) == ("64_lone", 0) and down(3612, 1200, 4296) == ("64_lone", 0)    # 260 and 290 tiles
    for rows, d, I in ((2400, 3216, 9248), (2068, 3776, 12760), (4895, 1584, 5296)):                  # 494 to 510
        assert down(rows, d, I) == ("128", 0), (rows, d, I)
    assert down(1264, 3224, 8544) == ("64_lone", 0) and down(2508, 1568, 3936) == ("64_lone", 0)      # every second row on a line
    for rows, d, I in ((2038, 2088, 6240), (2356, 1800, 5664)):                                       # and more than four rounds
        assert down(rows, d, I) == ("128", 0), (rows, d, I)
    assert down(1169, 3296, 11072) == ("128", 0)                                                      # all of them


def test_dx_of_later_chunks_of_few_rows_has_a_launch_of_its_own(mst):
    """Chunks of one row of large tiles whose weight gradients are read back: dX's long tiles would end that launch."""
    for d, I in ((4096, 14336), (4096, 11008), (3328, 12496)):
        for rows in (65, 100, 200, 256):
            assert mst.mst_mlp_dx_tile(rows, d, I, False) == "own", (rows, d, I)
    assert mst.mst_mlp_dx_tile(300, 4096, 14336, False) == "128"
    assert mst.mst_mlp_dx_tile(208, 5120, 13824, False) == "128"      # more 64 x 64 tiles than compute units


def test_dx_takes_128_by_128_tiles_only_where_it_is_waited_for(mst):
    """They cost 1.4 times the compute unit time: not in long chunks with as much other work, nor in short later chunks for
    which a launch of its own is estimated cheaper (each timed both ways, slower with them)."""
    tiles = lambda *shape: [g["dx_tile_rows"] for g in mst.mst_mlp_bwd_groups(*shape)]
    assert 128 not in tiles(16999, 1336, 4848, 7)[1:] and 128 not in tiles(6156, 2264, 6056, 4)
    assert 128 not in tiles(9576, 2016, 4232, 4) and 128 not in tiles(7788, 1952, 7584, 6)
    assert 128 not in tiles(1758, 776, 2808, 6) and 128 not in tiles(2170, 840, 3080, 5)
    assert tiles(2664, 1776, 6936, 3) == [128] * 3 and tiles(707, 1504, 5208, 1) == [128] == tiles(500, 4096, 14336, 1)


def test_workgroup_to_tile_map_is_a_bijection(mst):
    """Both maps of the 256 x 256 launches, on the host: every tile is the image of exactly one workgroup."""
    import ctypes
    lib = mst.load_mlp_library()
    s, f = ctypes.c_int32(), ctypes.c_int32()
    maps = set()
    for n_slow, n_fast in [(1, 1), (3, 5), (8, 4), (16, 4), (36, 6), (112, 16), (43, 7), (56, 16), (9, 33), (64, 8), (7, 100), (130, 2)]:
        grid = lib.mst_mlp_tile_grid(n_slow, n_fast)
        maps.add(grid == 8 * -(-n_slow * n_fast // 8))
        seen = set()
        for b in range(grid):
            rc = lib.mst_mlp_tile_of_workgroup(n_slow, n_fast, b, ctypes.byref(s), ctypes.byref(f))
            assert rc in (0, 1)
            if rc:
                assert 0 <= s.value < n_slow and 0 <= f.value < n_fast and (s.value, f.value) not in seen
                seen.add((s.value, f.value))
        assert len(seen) == n_slow * n_fast
    assert maps == {True, False}                     # padded super-tiles are among them
    assert lib.mst_mlp_tile_of_workgroup(4, 4, 10 ** 6, ctypes.byref(s), ctypes.byref(f)) == -1
    assert lib.mst_mlp_tile_of_workgroup(4, 4, 0, None, ctypes.byref(f)) == -1
    assert lib.mst_mlp_tile_grid(0, 4) == -1
