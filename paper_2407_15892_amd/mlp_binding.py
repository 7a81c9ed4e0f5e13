"""Thin ctypes binding of libmst_mlp.so: argument marshalling only.

Every step of the MLP path runs in the HIP kernels behind the C ABI declared in
include/mst_mlp.h.  PyTorch appears here only as the owner of device memory and
of the stream.  There is no CPU fallback: without the built library the calls
fail loudly.
"""
from __future__ import annotations

import ctypes
import os

from .binding import MST_OK, MstError, _ptr, _stream_handle
from .binding import load_library as _load_lmhead_library

HERE = os.path.dirname(os.path.abspath(__file__))
MLP_LIB_PATH = os.path.join(HERE, "libmst_mlp.so")

MLP_PROFILE_KINDS = 6

_lib = None


def load_mlp_library() -> ctypes.CDLL:
    """Load the in-tree MLP library (built by paper_2407_15892_amd.build.build)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(MLP_LIB_PATH):
        raise RuntimeError(
            f"{MLP_LIB_PATH} is missing: build it first (python -m paper_2407_15892_amd.build); "
            "there is no fallback path")
    _load_lmhead_library()      # loads PyTorch's HIP runtime globally first; also provides mst_strerror
    lib = ctypes.CDLL(MLP_LIB_PATH)
    c = ctypes
    lib.mst_mlp_version.restype = c.c_char_p
    lib.mst_mlp_version.argtypes = []
    lib.mst_mlp_workspace_bytes.restype = c.c_int
    lib.mst_mlp_workspace_bytes.argtypes = [c.c_int64, c.c_int64, c.c_int64, c.c_int32,
                                            c.POINTER(c.c_size_t), c.POINTER(c.c_size_t)]
    lib.mst_mlp_suggest_m.restype = c.c_int32
    lib.mst_mlp_suggest_m.argtypes = [c.c_int64, c.c_int64, c.c_int64]
    lib.mst_mlp_fwd.restype = c.c_int
    lib.mst_mlp_fwd.argtypes = [c.c_void_p] * 4 + [c.c_int64, c.c_int64, c.c_int64, c.c_int32,
                                                   c.c_void_p, c.c_size_t, c.c_void_p, c.c_void_p]
    lib.mst_mlp_bwd.restype = c.c_int
    lib.mst_mlp_bwd.argtypes = [c.c_void_p] * 5 + [c.c_int64, c.c_int64, c.c_int64, c.c_int32,
                                                   c.c_void_p, c.c_size_t] + [c.c_void_p] * 5
    lib.mst_mlp_tile_info.restype = c.c_int
    lib.mst_mlp_tile_info.argtypes = [c.c_int64, c.c_int64, c.c_int64, c.POINTER(c.c_int64)]
    lib.mst_mlp_dx_tile.restype = c.c_int32
    lib.mst_mlp_dx_tile.argtypes = [c.c_int64, c.c_int64, c.c_int64, c.c_int32]
    lib.mst_mlp_dx_tile_rows.restype = c.c_int32
    lib.mst_mlp_dx_tile_rows.argtypes = [c.c_int64, c.c_int64, c.c_int64, c.c_int32]
    lib.mst_mlp_fwd_groups.restype = c.c_int64
    lib.mst_mlp_fwd_groups.argtypes = [c.c_int64, c.c_int64, c.c_int64, c.c_int32, c.c_size_t, c.c_int32, c.c_int64, c.POINTER(c.c_int64)]
    lib.mst_mlp_bwd_groups.restype = c.c_int64
    lib.mst_mlp_bwd_groups.argtypes = [c.c_int64, c.c_int64, c.c_int64, c.c_int32, c.c_int32, c.c_int64, c.POINTER(c.c_int64)]
    lib.mst_mlp_line_panels.restype = c.c_int32
    lib.mst_mlp_line_panels.argtypes = [c.c_int64, c.c_int64, c.c_int64]
    lib.mst_mlp_da_in_gateup.restype = c.c_int32
    lib.mst_mlp_da_in_gateup.argtypes = [c.c_int64, c.c_int64, c.c_int64]
    lib.mst_mlp_tile_grid.restype = c.c_int32
    lib.mst_mlp_tile_grid.argtypes = [c.c_int32, c.c_int32]
    lib.mst_mlp_tile_of_workgroup.restype = c.c_int32
    lib.mst_mlp_tile_of_workgroup.argtypes = [c.c_int32] * 3 + [c.POINTER(c.c_int32)] * 2
    lib.mst_mlp_profile_enable.restype = c.c_int
    lib.mst_mlp_profile_enable.argtypes = [c.c_int]
    lib.mst_mlp_profile_collect.restype = c.c_int
    lib.mst_mlp_profile_collect.argtypes = [c.POINTER(c.c_double), c.POINTER(c.c_int64), c.POINTER(c.c_int64)]
    lib.mst_mlp_profile_kind_name.restype = c.c_char_p
    lib.mst_mlp_profile_kind_name.argtypes = [c.c_int]
    _lib = lib
    return lib


def _check(status: int) -> None:
    if status != MST_OK:
        raise MstError(status, _load_lmhead_library().mst_strerror(status).decode())


def mst_mlp_version() -> str:
    return load_mlp_library().mst_mlp_version().decode()


def mst_mlp_workspace_bytes(S: int, d: int, I: int, M: int):
    """(fwd_bytes, bwd_bytes) as the C call reports them."""
    f, b = ctypes.c_size_t(0), ctypes.c_size_t(0)
    _check(load_mlp_library().mst_mlp_workspace_bytes(S, d, I, M, ctypes.byref(f), ctypes.byref(b)))
    return int(f.value), int(b.value)


def mst_mlp_workspace_bytes_status(S: int, d: int, I: int, M: int) -> int:
    f, b = ctypes.c_size_t(0), ctypes.c_size_t(0)
    return int(load_mlp_library().mst_mlp_workspace_bytes(S, d, I, M, ctypes.byref(f), ctypes.byref(b)))


def mst_mlp_suggest_m(S: int, d: int, I: int) -> int:
    """Chunk count of the paper's constant chunk size C = d."""
    return int(load_mlp_library().mst_mlp_suggest_m(S, d, I))


def mst_mlp_fwd(X, Wg, Wu, Wd, M: int, workspace, O, stream=None) -> None:
    """Enqueue the forward pass.  X bf16 [S,d], Wg/Wu bf16 [I,d], Wd bf16 [d,I]; O bf16 [S,d] is overwritten."""
    S, d = X.shape
    I = Wg.shape[0]
    _check(load_mlp_library().mst_mlp_fwd(
        _ptr(X), _ptr(Wg), _ptr(Wu), _ptr(Wd), S, d, I, M,
        _ptr(workspace), workspace.numel() * workspace.element_size(), _ptr(O), _stream_handle(stream)))


def mst_mlp_bwd(X, Wg, Wu, Wd, dO, M: int, workspace, dX, dWg, dWu, dWd, stream=None) -> None:
    """Enqueue the backward pass.  dX bf16 [S,d]; dWg, dWu fp32 [I,d]; dWd fp32 [d,I]; all fully overwritten."""
    S, d = X.shape
    I = Wg.shape[0]
    _check(load_mlp_library().mst_mlp_bwd(
        _ptr(X), _ptr(Wg), _ptr(Wu), _ptr(Wd), _ptr(dO), S, d, I, M,
        _ptr(workspace), workspace.numel() * workspace.element_size(),
        _ptr(dX), _ptr(dWg), _ptr(dWu), _ptr(dWd), _stream_handle(stream)))


MLP_TILES = ("256", "128", "128_lone", "64", "64_lone", "64_long", "32", "128x256")     # MST_MLP_TILE_*


def mst_mlp_tile_info(rows: int, d: int, I: int) -> dict:
    """What a group of `rows` rows runs with: per product (tile, leading columns that large tiles take in a launch of their
    own, large tiles in super-tiles), and for the weight gradients (tile, dealt out evenly)."""
    a = (ctypes.c_int64 * 14)()
    _check(load_mlp_library().mst_mlp_tile_info(rows, d, I, a))
    out = {name: (MLP_TILES[a[3 * i]], int(a[3 * i + 1]), bool(a[3 * i + 2]))
           for i, name in enumerate(("gateup", "down", "da", "dx"))}
    out["dw"] = (MLP_TILES[a[12]], bool(a[13]))
    return out


MLP_DX_TILES = ("own", "256", "128", "64", "32")     # MST_MLP_DX_*


def mst_mlp_dx_tile(rows: int, d: int, I: int, first: bool) -> str:
    """How dX of a group of rows is computed: in a launch of its own, or by that of the weight gradients with this tile."""
    return MLP_DX_TILES[load_mlp_library().mst_mlp_dx_tile(rows, d, I, int(first))]


def mst_mlp_dx_tile_rows(rows: int, d: int, I: int, first: bool) -> int:
    """Rows of that tile, 0 where dX has a launch of its own."""
    return load_mlp_library().mst_mlp_dx_tile_rows(rows, d, I, int(first))


def mst_mlp_da_in_gateup(rows: int, d: int, I: int) -> bool:
    """Whether dA of a group of rows is computed by the launch of gate/up's backward."""
    return load_mlp_library().mst_mlp_da_in_gateup(rows, d, I) == 1


def mst_mlp_fwd_groups(S: int, d: int, I: int, M: int, workspace_bytes=None, output_overlaps: bool = False) -> list:
    """The groups of rows a forward call takes, as (rows, A in the rows of O behind the group).  workspace_bytes: of the
    workspace handed in (default: as many as the call needs)."""
    if workspace_bytes is None:
        workspace_bytes = mst_mlp_workspace_bytes(S, d, I, M)[0]
    lib = load_mlp_library()
    n = lib.mst_mlp_fwd_groups(S, d, I, M, workspace_bytes, int(output_overlaps), 0, None)
    a = (ctypes.c_int64 * (2 * max(n, 0)))()
    lib.mst_mlp_fwd_groups(S, d, I, M, workspace_bytes, int(output_overlaps), max(n, 0), a)
    return [(int(a[2 * i]), bool(a[2 * i + 1])) for i in range(n)]


def mst_mlp_bwd_groups(S: int, d: int, I: int, M: int, dx_overlaps: bool = False) -> list:
    """The groups of rows a backward call takes, each as a dict: its rows, how many of dG, dU and A are in dX, how dX is computed
    and the rows of its tile, whether dA is by the launch of gate/up's backward, the tile of the weight gradients."""
    lib = load_mlp_library()
    n = lib.mst_mlp_bwd_groups(S, d, I, M, int(dx_overlaps), 0, None)
    a = (ctypes.c_int64 * (6 * max(n, 0)))()
    lib.mst_mlp_bwd_groups(S, d, I, M, int(dx_overlaps), max(n, 0), a)
    return [{"rows": int(r[0]), "in_dx": int(r[1]), "dx": MLP_DX_TILES[r[2]], "dx_tile_rows": int(r[3]), "da_in_gateup": bool(r[4]),
             "dw": MLP_TILES[r[5]]} for r in (a[6 * i:6 * i + 6] for i in range(n))]


MLP_LINES = ("down", "da", "dx")     # MST_MLP_LINES_*


def mst_mlp_line_panels(rows: int, d: int, I: int) -> set:
    """The products that load rows which are not whole cache lines line by line."""
    mask = load_mlp_library().mst_mlp_line_panels(rows, d, I)
    return {name for i, name in enumerate(MLP_LINES) if mask >> i & 1}


def mst_mlp_profile_enable(every) -> None:
    """0 / False: off; n >= 1 (True = 1): bracket every n-th launch of each kernel kind with events."""
    _check(load_mlp_library().mst_mlp_profile_enable(int(every)))


def mst_mlp_profile_collect():
    """{kind name: (ms of the timed launches, timed launches, all launches)} since the last collect."""
    ms = (ctypes.c_double * MLP_PROFILE_KINDS)()
    n = (ctypes.c_int64 * MLP_PROFILE_KINDS)()
    issued = (ctypes.c_int64 * MLP_PROFILE_KINDS)()
    _check(load_mlp_library().mst_mlp_profile_collect(ms, n, issued))
    lib = load_mlp_library()
    return {lib.mst_mlp_profile_kind_name(i).decode(): (float(ms[i]), int(n[i]), int(issued[i])) for i in range(MLP_PROFILE_KINDS)}
