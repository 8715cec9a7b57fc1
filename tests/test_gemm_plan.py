"""The GEMM's plan, on the host: the shapes of the GPU tests reach every tile config of every
epilogue, and a plan keeps what the kernel and its buffers need."""
import ctypes

import pytest

from paper_2608_11235_amd import _lib
from tests.test_gpu_gemm_tiles import HEAD_BLOCKS, HEADS, SHAPES

CUS = 256
CONFIGS = set(range(10))


class Plan(ctypes.Structure):
    _fields_ = [("cfg", ctypes.c_int), ("tiles", ctypes.c_int), ("splits", ctypes.c_int),
                ("ws_floats", ctypes.c_size_t)]


def _plan(M, N, K):
    f = _lib.load()._ZN4cora9gemm_planEiiii
    f.restype, f.argtypes = Plan, [ctypes.c_int] * 4
    return f(M, N, K, CUS)


def _split_plan(M, N, K, splits, fold_us):
    f = _lib.load()._ZN4cora15gemm_plan_splitEiiiiid
    f.restype, f.argtypes = Plan, [ctypes.c_int] * 5 + [ctypes.c_double]
    return f(M, N, K, CUS, splits, fold_us)


def _layer_configs(bl, d, H, Hkv, hd, ffn):
    """(epilogue, config) of the four GEMMs of a layer whose batch is the planned one."""
    M, f_pad = bl[0] * bl[1], -(-ffn // 64) * 64
    p = _split_plan(M, (H + 2 * Hkv) * hd, d, 0, 7.0)
    yield ("qkv" if p.splits == 1 else "partial"), p.cfg
    for K in (H * hd, f_pad):
        p = _split_plan(M, d, K, 0, 0.0)
        yield ("residual" if p.splits == 1 else "partial"), p.cfg
    yield "swiglu", _plan(M, 2 * f_pad, d).cfg


def test_layer_shapes_reach_every_config_of_every_epilogue():
    seen = {c for s in SHAPES for c in _layer_configs(*s)}
    for epilogue in ("qkv", "residual", "partial", "swiglu"):
        assert {c for e, c in seen if e == epilogue} == CONFIGS, epilogue


def test_head_shapes_reach_every_config():
    assert {_plan(B * blk, vocab, 384).cfg for B, blk, vocab in HEAD_BLOCKS} == CONFIGS
    assert {_plan(rows, vocab, 256).cfg for rows, vocab in HEADS} == CONFIGS - {2, 3}


@pytest.mark.parametrize("fold_us", [0.0, 7.0])
def test_split_count_holds_for_fewer_rows(fold_us):
    """The split count planned for a full batch is a plan for every smaller one, within the
    workspace, and K divides into pairs of slices."""
    for M in (1, 40, 64, 65, 109, 512, 1280, 4096):
        for N, K in ((64, 64), (768, 3584), (3584, 3584), (4096, 12288), (4608, 3584), (8192, 28672)):
            splits = _split_plan(M, N, K, 0, fold_us).splits
            assert K % (64 * splits) == 0
            for live in {1, max(1, M // 8), max(1, M // 2), M}:
                p = _split_plan(live, N, K, splits, fold_us)
                assert p.splits == splits and p.tiles > 0
                assert p.ws_floats <= 2 * CUS * 256 * 256
                assert p.ws_floats == (0 if splits == 1 else splits * live * N)
