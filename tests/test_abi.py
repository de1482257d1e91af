"""The C-ABI library loads, exports every entry point the header declares, and
rejects bad arguments on the host (no device work is needed for these)."""
import ctypes
import os

import pytest

from paper_2512_22420_amd import binding as nb
from paper_2512_22420_amd import workload as W
from paper_2512_22420_amd.device import model_desc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "nightjar.h")

pytestmark = pytest.mark.skipif(not os.path.exists(nb.LIB_PATH), reason="libnightjar.so not built")


def test_exports_every_declared_function():
    import glob
    names = nb.header_functions(HEADER)
    assert "nightjar_verify_step" in names and "nightjar_kv_append" in names
    headers = sorted(glob.glob(os.path.join(ROOT, "include", "*.h")))
    assert len(headers) >= 2
    L = nb.lib()
    for h in headers:
        for n in nb.header_functions(h):
            assert hasattr(L, n), (h, n)
            assert n in nb._SIGS, (h, n)  # the binding declares it too


def test_struct_sizes_match_header_layout():
    assert ctypes.sizeof(nb.ModelDesc) == 11 * 4
    assert ctypes.sizeof(nb.LayerWeights) == 6 * 8
    assert ctypes.sizeof(nb.Weights) == 4 * 8
    assert ctypes.sizeof(nb.KvCache) == 3 * 8


def test_workspace_bytes_monotone_and_validating():
    d = model_desc(W.LLAMA8B_LAYER)
    small = nb.workspace_bytes(d, 1, 0)
    big = nb.workspace_bytes(d, 8, 5)
    assert 0 < small < big
    assert big % 256 == 0
    with pytest.raises(nb.NightjarError):
        nb.workspace_bytes(d, 1, 16)  # the window must fit one 16-token block
    bad = model_desc(W.LLAMA8B_LAYER)
    bad.block_size = 32
    assert nb.lib().nightjar_workspace_bytes(ctypes.byref(bad), 1, 0) == 0
    assert "block_size" in nb.last_error()
    bad = model_desc(W.LLAMA8B_LAYER)
    bad.n_kv_heads = 5
    assert nb.lib().nightjar_workspace_bytes(ctypes.byref(bad), 1, 0) == 0


def test_verify_step_rejects_bad_arguments_on_host():
    d = model_desc(W.TINY_F32)
    w = nb.Weights()
    kv = nb.KvCache()
    rc = nb.lib().nightjar_verify_step(ctypes.byref(d), ctypes.byref(w), ctypes.byref(kv), 0, 1, 0, 0, 0, 0, 0,
                                       2, 3, 0, 0, 0, 0, 0, 0)
    assert rc == nb.NJ_EINVAL and "weights" in nb.last_error()
    rc = nb.lib().nightjar_verify_step(None, ctypes.byref(w), ctypes.byref(kv), 0, 1, 0, 0, 0, 0, 0,
                                       2, 3, 0, 0, 0, 0, 0, 0)
    assert rc == nb.NJ_EINVAL and "desc" in nb.last_error()
    rc = nb.lib().nightjar_verify_step(ctypes.byref(d), ctypes.byref(w), ctypes.byref(kv), 0, 1, 0, 0, 0, 0, 0,
                                       2, 16, 0, 0, 0, 0, 0, 0)
    assert rc == nb.NJ_EINVAL and "k must be" in nb.last_error()


def test_gemm_rejects_bad_shapes_on_host():
    L = nb.lib()
    big = 1 << 30
    assert L.nightjar_gemm(nb.NJ_BF16, 16, 16, 16, 4, 32, 40, nb.NJ_GEMM_STORE, 256, big, 0) == nb.NJ_EINVAL  # K % 32
    assert L.nightjar_gemm(nb.NJ_BF16, 16, 16, 16, 4, 24, 64, nb.NJ_GEMM_STORE, 256, big, 0) == nb.NJ_EINVAL  # N % 16
    assert L.nightjar_gemm(nb.NJ_BF16, 16, 16, 16, 4, 30, 64, nb.NJ_GEMM_SWIGLU, 256, big, 0) == nb.NJ_EINVAL
    assert L.nightjar_gemm(nb.NJ_BF16, 0, 16, 16, 4, 32, 64, nb.NJ_GEMM_STORE, 256, big, 0) == nb.NJ_EINVAL
    assert L.nightjar_gemm(nb.NJ_BF16, 16, 16, 16, 0, 32, 64, nb.NJ_GEMM_STORE, 256, big, 0) == nb.NJ_EINVAL
    assert L.nightjar_gemm(7, 16, 16, 16, 1, 32, 64, nb.NJ_GEMM_STORE, 256, big, 0) == nb.NJ_EINVAL
    # a workspace smaller than the split-K scratch is refused before any launch
    need = nb.gemm_workspace_bytes(nb.NJ_BF16, 48, 4096, 14336, nb.NJ_GEMM_RESIDUAL)
    assert need > 256
    assert L.nightjar_gemm(nb.NJ_BF16, 16, 16, 16, 48, 4096, 14336, nb.NJ_GEMM_RESIDUAL, 256, need - 256, 0) == nb.NJ_EINVAL
    assert "workspace" in nb.last_error()


def test_kv_append_requires_a_preceding_verify_step():
    d = model_desc(W.TINY_F32)
    ptrs = (ctypes.c_void_p * 1)(16)
    kv = nb.KvCache(ctypes.cast(ptrs, ctypes.POINTER(ctypes.c_void_p)), ctypes.cast(ptrs, ctypes.POINTER(ctypes.c_void_p)), 4)
    rc = nb.lib().nightjar_kv_append(ctypes.byref(d), ctypes.byref(kv), 16, 4, 16, 16, 2, 3, 256, 1 << 20, 0)
    assert rc == nb.NJ_EINVAL and "no verify step" in nb.last_error()


def test_gemm_with_plan_rejects_impossible_plans_on_host():
    L = nb.lib()
    ws = 1 << 30
    st = nb.NJ_GEMM_STORE
    # tiled kernels need K % 64 == 0
    assert L.nightjar_gemm_with_plan(nb.NJ_BF16, 16, 16, 16, 200, 256, 96, st, nb.NJ_GEMM_TILE_128x128, 0, 256, ws, 0) \
        == nb.NJ_EINVAL
    assert "K % 64" in nb.last_error()
    # a run that cuts tiles between workgroups may have at most 1024 of them
    assert nb.lib().nightjar_gemm_plan_workspace_bytes(nb.NJ_BF16, 768, 128256, 4096, st, nb.NJ_GEMM_TILE_128x128, 2) == 0
    assert "at most 1024 workgroups" in nb.last_error()
    assert nb.lib().nightjar_gemm_plan_workspace_bytes(nb.NJ_BF16, 768, 4096, 4096, st, nb.NJ_GEMM_TILE_128x128,
                                                       -1100) == 0
    # stream-K grids: tiled kernels only, and not the 256x256 tile
    assert nb.lib().nightjar_gemm_plan_workspace_bytes(nb.NJ_BF16, 768, 4096, 4096, st, nb.NJ_GEMM_TILE_256x256,
                                                       -100) == 0
    assert "256x256" in nb.last_error()
    assert nb.lib().nightjar_gemm_plan_workspace_bytes(nb.NJ_BF16, 768, 4096, 4096, st, nb.NJ_GEMM_TILE_128x256,
                                                       -100) > 0
    # a grid of 3 x 12 workgroups on 12 tiles is a plain 3-way split, which the 256x256 tile runs
    assert nb.lib().nightjar_gemm_plan_workspace_bytes(nb.NJ_BF16, 768, 1024, 4096, st, nb.NJ_GEMM_TILE_256x256,
                                                       -36) > 0
    # auto plan takes no split; fp32 has one kernel; bad kernel id
    assert L.nightjar_gemm_plan_workspace_bytes(nb.NJ_BF16, 64, 256, 256, st, nb.NJ_GEMM_AUTO, 2) == 0
    assert L.nightjar_gemm_plan_workspace_bytes(nb.NJ_F32, 64, 256, 256, st, nb.NJ_GEMM_STREAM, 0) == 0
    assert L.nightjar_gemm_plan_workspace_bytes(nb.NJ_BF16, 64, 256, 256, st, nb.NJ_GEMM_TILE_96x128 + 1, 0) == 0
    assert L.nightjar_gemm_plan_workspace_bytes(nb.NJ_BF16, 64, 256, 256, st, nb.NJ_GEMM_STREAM, -1) == 0
    # the workspace grows with the split (fp32 partials per chunk)
    a = nb.gemm_plan_workspace_bytes(nb.NJ_BF16, 384, 4096, 4096, st, nb.NJ_GEMM_TILE_256x256, 1)
    b = nb.gemm_plan_workspace_bytes(nb.NJ_BF16, 384, 4096, 4096, st, nb.NJ_GEMM_TILE_256x256, 4)
    assert b >= a + 4 * 384 * 4096 * 4
    # a workspace one byte short is refused before any launch
    assert L.nightjar_gemm_with_plan(nb.NJ_BF16, 16, 16, 16, 384, 4096, 4096, st, nb.NJ_GEMM_TILE_256x256, 4, 256,
                                     b - 1, 0) == nb.NJ_EINVAL


def test_gemm_partials_lie_past_the_counters_of_every_shape():
    """Calls of different shapes may share a workspace: a split plan's partial
    sums start past the region in which any plan keeps its counters (1024 of
    256 bytes, behind the 256-byte error word), not right behind its own."""
    counters, res = 256 + 1024 * 256, nb.NJ_GEMM_RESIDUAL
    for kernel, split, M, N, K in [(nb.NJ_GEMM_STREAM, 2, 16, 128, 4096), (nb.NJ_GEMM_STREAM, 8, 39, 4096, 14336),
                                   (nb.NJ_GEMM_TILE_128x128, 4, 160, 4096, 14336), (nb.NJ_GEMM_TILE_96x128, 2, 96, 128, 512)]:
        need = nb.gemm_plan_workspace_bytes(nb.NJ_BF16, M, N, K, res, kernel, split)
        assert need >= counters + split * M * N * 4, (kernel, split, M, N, K, need)
    # the planner's own choice for the 8B down projection at 39 rows splits K
    need = nb.gemm_workspace_bytes(nb.NJ_BF16, 39, 4096, 14336, res)
    assert need >= counters + 2 * 39 * 4096 * 4
    assert nb.gemm_plan_workspace_bytes(nb.NJ_BF16, 39, 4096, 14336, res, nb.NJ_GEMM_AUTO, 0) == need


@pytest.mark.parametrize("M,N,K,epi", [
    (160, 28672, 4096, nb.NJ_GEMM_SWIGLU), (2048, 37888, 3584, nb.NJ_GEMM_SWIGLU), (305, 128256, 4096, nb.NJ_GEMM_STORE),
    (256, 28672, 512, nb.NJ_GEMM_STORE), (8, 4096, 4096, nb.NJ_GEMM_RESIDUAL)])
def test_gemm_without_split_needs_no_scratch(M, N, K, epi):
    """A plan that does not split K keeps nothing in the workspace, so such calls
    may overlap on one: all that is asked for is the 256 bytes of the error word."""
    assert nb.gemm_workspace_bytes(nb.NJ_BF16, M, N, K, epi) == 256


def test_gemm_plan_info():
    res = nb.NJ_GEMM_RESIDUAL
    assert nb.gemm_plan_info(nb.NJ_F32, 4, 50, 70, res, nb.NJ_GEMM_AUTO, 0)["kernel"] == "f32"
    small = nb.gemm_plan_info(nb.NJ_BF16, 8, 4096, 14336, res, nb.NJ_GEMM_AUTO, 0)
    assert small == {"kernel": "small", "tile": (16, 16), "chunks": 1, "workgroups": 256, "stream_k": False}
    stream = nb.gemm_plan_info(nb.NJ_BF16, 48, 4096, 14336, res, nb.NJ_GEMM_STREAM, 4)
    assert stream == {"kernel": "stream", "tile": (48, 128), "chunks": 4, "workgroups": 128, "stream_k": False}
    tile = nb.gemm_plan_info(nb.NJ_BF16, 768, 4096, 14336, res | nb.NJ_GEMM_KBLOCKED, nb.NJ_GEMM_TILE_128x256, -200)
    assert tile["kernel"] == "tile" and tile["tile"] == (128, 256) and tile["stream_k"] and tile["workgroups"] == 198
    for M in (160, 320, 600, 2048):  # the 320x256 tile runs whole sums only
        for N, K in ((128256, 4096), (37888, 3584), (4096, 14336)):
            p = nb.gemm_plan_info(nb.NJ_BF16, M, N, K, nb.NJ_GEMM_STORE, nb.NJ_GEMM_AUTO, 0)
            assert p["tile"] != (320, 256) or (p["chunks"] == 1 and not p["stream_k"])
    with pytest.raises(nb.NightjarError):
        nb.gemm_plan_info(nb.NJ_BF16, 64, 256, 256, res, nb.NJ_GEMM_AUTO, 2)
    assert nb.lib().nightjar_gemm_plan_info(nb.NJ_BF16, 64, 256, 256, res, nb.NJ_GEMM_AUTO, 0, None) == nb.NJ_EINVAL


@pytest.mark.parametrize("M,N,K,kernel", [
    (8, 4096, 14336, "small"), (9, 4096, 14336, "stream"), (16, 3584, 18944, "stream"), (16, 2048, 8192, "stream"),
    (16, 4096, 6144, "small"), (9, 4096, 6176, "stream")])
def test_row_major_residual_of_long_k_streams_past_8_rows(M, N, K, kernel):
    """There the small-window kernel's reads of row-major x cost more than its K split saves."""
    assert nb.gemm_plan_info(nb.NJ_BF16, M, N, K, nb.NJ_GEMM_RESIDUAL, nb.NJ_GEMM_AUTO, 0)["kernel"] == kernel


def test_stage_entries_reject_bad_arguments_on_host():
    desc = model_desc(W.QWEN7B)  # G = 7: k = 9 gives 70 query rows per KV head
    n = nb.attn_workspace_bytes(desc, 1, 9)
    rc = nb.lib().nightjar_attn_verify(ctypes.byref(desc), 16, 16, 16, 4, 16, 16, 16, 4, 16, 1, 9, 16, 256, n, 0)
    assert rc == nb.NJ_EINVAL and "64 query rows" in nb.last_error()
    rc = nb.lib().nightjar_attn_verify(ctypes.byref(desc), 16, 16, 16, 4, 16, 16, 16, 4, 16, 1, 2, 16, 256, 255, 0)
    assert rc == nb.NJ_EINVAL and "workspace" in nb.last_error()
    rc = nb.lib().nightjar_attn_verify(ctypes.byref(desc), 0, 16, 16, 4, 16, 16, 16, 4, 16, 1, 2, 16, 256, n, 0)
    assert rc == nb.NJ_EINVAL and "NULL" in nb.last_error()
    d8 = model_desc(W.LLAMA8B_LAYER)
    m = nb.rmsnorm_rope_workspace_bytes(d8, 2, 3)
    assert m > nb.rmsnorm_rope_workspace_bytes(d8, 1, 3) > 0
    rc = nb.lib().nightjar_rmsnorm_rope(ctypes.byref(d8), 16, 16, 16, 16, 2, 3, 16, 16, 8, 256, m, 0)
    assert rc == nb.NJ_EINVAL and "aligned" in nb.last_error()
    rc = nb.lib().nightjar_rmsnorm_rope(ctypes.byref(d8), 16, 16, 16, 16, 2, 16, 16, 16, 16, 256, m, 0)
    assert rc == nb.NJ_EINVAL


@pytest.mark.parametrize("shape,max_B,max_k", [(W.LLAMA8B_LAYER, 128, 5), (W.QWEN7B, 256, 7), (W.LLAMA1B_DRAFT, 64, 4)],
                         ids=["8b-layer", "qwen7b", "1b-draft"])
def test_max_workspace_serves_every_smaller_window(shape, max_B, max_k):
    """nightjar_workspace_bytes(max_B, max_k) is enough for every (B, k) below
    it, whatever GEMM plan (split partials included) the smaller window picks."""
    L = nb.lib()
    d = model_desc(shape)
    top = L.nightjar_workspace_bytes(ctypes.byref(d), max_B, max_k)
    assert top > 0
    Bs = sorted(set(list(range(1, 17)) + list(range(16, max_B + 1, 7)) + [max_B]))
    for B in Bs:
        for k in range(max_k + 1):
            need = L.nightjar_workspace_bytes(ctypes.byref(d), B, k)
            assert 0 < need <= top, (B, k, need, top)
