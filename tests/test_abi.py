"""The C-ABI library loads and exports every symbol include/rv.h declares (no compute)."""
import ctypes
import os
import re

from paper_2401_01728_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared(header="rv.h"):
    text = open(os.path.join(ROOT, "include", header)).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(rv_[a-z0-9_]+)\s*\(", text)))


def test_header_and_binding_agree():
    assert _declared() == sorted(_lib.SYMBOLS)
    assert _declared("rv_kernels.h") == sorted(_lib.KERNEL_SYMBOLS)


def test_library_exports_every_symbol():
    lib = _lib.lib()
    for name in _declared() + _declared("rv_kernels.h"):
        assert getattr(lib, name) is not None


def test_argument_validation_needs_no_device():
    lib = _lib.lib()
    INVAL = -1
    assert lib.rv_cluster_average(None, 2, 8, 1, None, 1, None, 0, 0.0, None) == INVAL
    arr = (ctypes.c_void_p * 2)(16, 32)
    assert lib.rv_cluster_average(arr, 0, 8, 1, None, 1, None, 0, 0.0, None) == INVAL     # C < 1
    assert lib.rv_cluster_average(arr, 2, 8, 0, None, 1, None, 0, 0.0, None) == INVAL     # R < 1
    assert lib.rv_cluster_average(arr, 2, 0, 1, None, 1, None, 0, 0.0, None) == INVAL     # n == 0
    assert lib.rv_cluster_average(arr, 2, 8, 1, None, 0, None, 0, 0.0, None) == INVAL     # no output
    assert lib.rv_cluster_average(arr, 2, 8, 1, None, 1, 64, 2, 0.0, None) == INVAL       # grad_replica
    same = (ctypes.c_void_p * 2)(16, 16)
    assert lib.rv_cluster_average(same, 2, 8, 1, None, 1, None, 0, 0.0, None) == INVAL    # aliasing
    assert lib.rv_block_update(None, 16, 4, 0.1, None, None) == INVAL
    assert lib.rv_stage_create(None, None) == INVAL
    dims = (ctypes.c_int64 * 3)(4, 0, 3)
    d = _lib.StageDesc(0, 0, 2, dims, 8, 1, 0.1, 1e-5, None)
    h = ctypes.c_void_p()
    assert lib.rv_stage_create(ctypes.byref(d), ctypes.byref(h)) == INVAL                 # zero width
    d = _lib.StageDesc(0, 1, 2, dims, 8, 1, 0.1, 1e-5, None)
    assert lib.rv_stage_create(ctypes.byref(d), ctypes.byref(h)) == INVAL                 # MLP must be fp32
    d = _lib.StageDesc(0, 0, 2, dims, 8, -1, 0.1, 1e-5, None)
    assert lib.rv_stage_create(ctypes.byref(d), ctypes.byref(h)) == INVAL                 # tau < 0
    assert lib.rv_stage_num_params(None) == 0
    assert lib.rv_strerror(-2).decode().startswith("tau+1")


def test_large_products_are_not_cut():
    """From 64 tiles of 256x256 on no product is cut into stretches (a step needs the CU time for its other streams); at the
    sizes that the rule's comment quotes the forms are those."""
    def form(M, N, K):
        tile, parts = ctypes.c_int(), ctypes.c_int()
        assert _lib.lib().rv_k_gemm_part_form(M, N, K, ctypes.byref(tile), ctypes.byref(parts)) == 0
        return tile.value, parts.value
    for tm, tn in ((8, 8), (4, 16), (5, 13), (16, 4), (11, 6), (18, 16), (64, 16)):
        for M in (256 * tm - 192, 256 * tm):
            for N in (256 * tn - 192, 256 * tn):
                for K in (N, 2 * N, 3 * N, 4 * N):
                    assert form(M, N, K) == (0, 1), (M, N, K)
    for shape, want in (((64, 2048, 8192), (1064, 8)), ((128, 1024, 4096), (1032, 4)), ((1024, 2048, 8192), (1128, 2)),
                        ((1152, 1600, 6400), (1128, 2)), ((256, 448, 1792), (1032, 4))):
        assert form(*shape) == want
    assert _lib.lib().rv_k_gemm_part_form(64, 64, 64, None, None) == -1
