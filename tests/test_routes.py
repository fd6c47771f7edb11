"""The kernels that calls of the C ABI launch (host side only: tests/record.py
records the launches of the built library on 256 compute units)."""
import re

import pytest

import paper_2406_02528_amd as mmf
import test_gpu_ragged
import test_gpu_skinny
from record import AUTO, GEMM, GEMV, call, kernels, record  # noqa: F401

A = 0x100000000  # made-up 256-byte aligned device address, never dereferenced
BIG = 1 << 40


def bwd(M, K, N, ws=A):
    return call("mmf_bitlinear_bwd", A, A, 0, A, A, A, A, A, A, A, A, A, A, M, K, N, ws, BIG, None)


def test_backward_of_very_many_tokens_launches():
    """2^24 token rows and more of a dO that needs padding: every launch stays
    inside the runtime's limit of 2^32 threads."""
    for r in record([bwd((1 << 24) + 7, 16, 3), bwd(1 << 25, 16, 60)]):
        assert r["status"] == 0 and kernels(r)[0] == "pad_rows_kernel"


# Calls whose form depends on the process-wide path: M of 8 and 20 rows fit the
# fused decode kernel, 45 and 300 do not (K = 2048), with and without scratch.
def _path_calls(M, **kw):
    K, N, d = 2048, 6144, 2048
    return [call("mmf_bitlinear_fwd", A, A, A, A, A, M, K, N, None, **kw),
            call("mmf_bitlinear_fwd_ws", A, 0, A, A, A, A, M, K, N, A, BIG, None, **kw),
            call("mmf_bitlinear_fwd_noalloc", A, 0, A, A, A, A, M, K, N, None, **kw),
            call("mmf_bitlinear_fwd_bias", A, 0, A, A, A, A, A, M, K, N, None, **kw),
            call("mmf_glu_fwd", A, A, A, A, A, M, K, N // 2, None, **kw),
            call("mmf_mlgru_fwd", A, 0, A, A, A, A, A, A, A, A, A, A, A, A, M, 1, d, None, 0, None, **kw),
            call("mmf_ternary_gemm_dequant", A, A, A, A, A, A, M, K, N, None, **kw)]


@pytest.mark.parametrize("capture", [False, True])
@pytest.mark.parametrize("path,other", [(AUTO, GEMM), (AUTO, GEMV), (GEMV, AUTO), (GEMM, GEMV)])
def test_a_path_set_meanwhile_does_not_reach_a_running_call(path, other, capture):
    """Another thread's mmf_set_path during a call leaves that call as it was:
    the same kernels, and scratch wherever act-quant writes."""
    Ms, ns = (8, 20, 45, 300), range(1, 6)
    out = record([c for M in Ms for n in (0, *ns) for c in _path_calls(M, path=path, capture=capture, switch=(n, other))])
    per = len(_path_calls(1))
    for i in range(len(Ms)):
        runs = [out[(i * (len(ns) + 1) + n) * per:][:per] for n in (0, *ns)]
        for got in runs:  # the first one is undisturbed
            for w, g in zip(runs[0], got):
                assert w["launches"]
                assert [(x["kernel"], x["grid"]) for x in g["launches"]] == [(x["kernel"], x["grid"]) for x in w["launches"]]
                assert (g["status"], g["allocs"], g["frees"]) == (0, w["allocs"], w["allocs"])
                assert all(x["args"][2] >= A for x in g["launches"] if x["kernel"].startswith("act_quant_kernel"))


def _alloc_calls(M, K, **kw):
    N = 1024
    # the fused kernel takes 16 rows up to K = 2048 in bf16, 1024 in float32
    f32 = [call("mmf_bitlinear_fwd_f32", A, A, A, A, A, M, K, N, None, **kw)] if K <= 1024 else []
    return f32 + [call("mmf_bitlinear_fwd", A, A, A, A, A, M, K, N, None, **kw),
                  call("mmf_bitlinear_fwd_noalloc", A, 0, A, A, A, A, M, K, N, None, **kw),
                  call("mmf_bitlinear_fwd_bias", A, 0, A, A, A, A, A, M, K, N, None, **kw),
                  call("mmf_glu_fwd", A, A, A, A, A, M, K, N // 2, None, **kw)]


@pytest.mark.parametrize("M,K", [(1, 2048), (16, 2048), (17, 16), (20, 2048), (32, 1024), (32, 2048)])
def test_few_tokens_without_workspace_allocate_nothing(M, K):
    """Forms without caller scratch run up to 32 tokens as fused decode
    launches: no allocation, which would cost more than the second launch, can
    fail, and cannot be captured everywhere."""
    for r in record([c for kw in ({}, {"fail_alloc": True}, {"capture": True}) for c in _alloc_calls(M, K, **kw)]):
        assert (r["status"], r["allocs"]) == (0, 0)
        assert kernels(r) == ["decode_kernel"] * -(-M // 16)


def test_calls_that_need_scratch_allocate_it():
    for M, K in ((17, 2064), (33, 2048), (65, 4096)):
        for r in record(_alloc_calls(M, K)):
            assert r["status"] == 0 and r["allocs"] == r["frees"] and kernels(r) == ["act_quant_kernel", "skinny_kernel"]
        failed = [r["status"] for r in record(_alloc_calls(M, K, fail_alloc=True))]
        assert failed == [5, 0, 5, 5]  # the second form's scratch is static


# Both sides of the line between the K-split and the tiled kernel, from x and
# from rows of q, as measured beside the rule in skinny.hip; the last ones are
# tall and narrow (K-split re-reads the rows in every column strip).
@pytest.mark.parametrize("K,N,split,tiled", [
    (1024, 1024, [17, 1024], [2048, 16384]), (2048, 2048, [64, 1024, 2048], [3072, 4096]),
    (2048, 6144, [32, 128, 384, 640], [768, 1024]), (2048, 11264, [33, 128, 320], [512]),
    (5120, 2048, [64, 1024, 2048], [3072, 4096]), (5120, 15360, [128, 256], [384, 512, 1536]),
    (2048, 2050, [256, 768], [2048]), (5120, 1024, [512], [8192]), (5120, 2050, [512], [16384]),
    (13824, 3000, [512], [12000]), (13824, 11264, [256, 384], [512]), (1024, 64, [40000], [65536])])
def test_few_rows_split_k_and_many_do_not(K, N, split, tiled):
    calls = [call("mmf_bitlinear_fwd_ws", A, 0, A, A, A, A, M, K, N, A, BIG, None) for M in split + tiled]
    assert [kernels(r)[-1] for r in record(calls)] == ["skinny_kernel"] * len(split) + ["gemm_kernel"] * len(tiled)


def test_decode_slices_give_way_to_the_k_split_kernel():
    """17 to 64 rows that the tiled kernel would not get anyway: with scratch
    (or from rows of q, which need none) never several decode launches."""
    shapes = [(17, 32, 58752), (28, 144, 61216), (32, 7680, 11264), (64, 5120, 27648), (17, 16, 16)]
    for r in record([call("mmf_bitlinear_fwd_ws", A, 0, A, A, A, A, *s, A, BIG, None) for s in shapes] +
                    [call("mmf_ternary_gemm_dequant", A, A, A, A, A, A, *s, None) for s in shapes]):
        assert kernels(r)[-1] == "skinny_kernel"


def _form(launch):
    """A skinny_kernel's row blocks x column blocks / steps in flight."""
    m = re.match(r"skinny_kernel<(\d+), (\d+), (\d+), (\d+), (\d+), ", launch["kernel"])
    return f"{m[1]}x{int(m[2]) * int(m[3]) * int(m[4])}/{m[5]}" if m else \
        {"gemm_kernel": "tiled", "decode_kernel": "decode"}[launch["kernel"].split("<")[0]]


@pytest.mark.parametrize("name", ["FORWARD", "RAW", "GLU", "GATES"])
def test_gpu_shapes_take_the_tiles_they_name(name):
    """The K-split tile forms that test_gpu_skinny.py names beside its shapes."""
    shapes = getattr(test_gpu_skinny, name)
    make = {"FORWARD": lambda M, K, N: call("mmf_bitlinear_fwd_ws", A, 0, A, A, A, A, M, K, N, A, BIG, None),
            "RAW": lambda M, K, N: call("mmf_ternary_gemm_i32", A, A, A, M, K, N, None),
            "GLU": lambda M, K, L: call("mmf_glu_fwd_ws", A, 0, A, A, A, A, M, K, L, A, BIG, None),
            "GATES": lambda M, K, d: call("mmf_mlgru_proj", A, 0, A, A, A, A, A, A, M, K, d, A, BIG, None)}[name]
    out = record([make(*s) for s in shapes])
    assert {s: _form(r["launches"][-1]) for s, r in zip(shapes, out)} == shapes


def test_gpu_dy_shapes_take_the_tiles_they_name():
    want = test_gpu_ragged.DY_TILES
    for (tile, r) in zip(want.values(), record([bwd(*s[:3]) for s in want])):
        assert [k["kernel"] for k in r["launches"] if k["kernel"].startswith("dy_kernel")] == \
            ["dy_kernel<unsigned short, DyTile<%d, %d> >" % tile]


@pytest.mark.parametrize("M,K,N", [
    (256, 1024, 1002), (257, 1024, 1002), (1937, 2288, 3998), (8192, 2048, 11266), (40, 512, 2304), (300, 1040, 2304),
    (2048, 2048, 6144), (2048, 2048, 1920), (4096, 1024, 8256), (8192, 2048, 11328), (1024, 5120, 15360)])
def test_tile_plan_names_the_tile_that_is_launched(M, K, N):
    """mmf_prefill_tile_plan against the launches of the tiled kernel, for every
    epilogue; a bias alone runs on the dequantising epilogue's tiles."""
    ws = (M, K, N, A, BIG, None)
    forms = {mmf.MMF_EPILOGUE_DEQUANT: [call("mmf_bitlinear_fwd_ws", A, 0, A, A, A, A, *ws, path=GEMM)],
             mmf.MMF_EPILOGUE_RAW_I32: [call("mmf_ternary_gemm_i32", A, A, A, M, K, N, None, path=GEMM)]}
    if N % 4 == 0:
        forms[mmf.MMF_EPILOGUE_DEQUANT].append(call("mmf_bitlinear_fwd_bias", A, 0, A, A, A, A, A, M, K, N, None, path=GEMM))
    if N % 32 == 0:
        forms[mmf.MMF_EPILOGUE_GLU] = [call("mmf_glu_fwd_ws", A, 0, A, A, A, A, M, K, N // 2, A, BIG, None, path=GEMM)]
    if N % 48 == 0:
        forms[mmf.MMF_EPILOGUE_AFFINE] = [
            call("mmf_mlgru_proj", A, 0, A, A, A, A, A, A, M, K, N // 3, A, BIG, None, path=GEMM)]
    for ep, calls in forms.items():
        plan = mmf.mmf_prefill_tile_plan(M, K, N, ep).removesuffix("_paired")
        for r in record(calls):
            assert r["status"] == 0
            assert re.match(r"gemm_kernel<(\d+), (\d+), ", r["launches"][-1]["kernel"]).groups() == tuple(plan.split("x"))


# One token per sequence through the mixer: where the recurrence runs.  Inside
# the output projection's decode launch where that takes the rows and the new
# state is an array of its own; with the state in place as its own launch;
# otherwise inside act-quant.
@pytest.mark.parametrize("B,in_place,want", [
    (1, False, ["decode_kernel", "decode_kernel"]), (16, False, ["decode_kernel", "act_quant_kernel", "skinny_kernel"]),
    (4, True, ["decode_kernel", "mlgru_apply_kernel", "decode_kernel"]),
    (17, False, ["act_quant_kernel", "skinny_kernel"] * 2), (17, True, ["act_quant_kernel", "skinny_kernel"] * 2)])
def test_decode_step_routes(B, in_place, want):
    h = A if in_place else 2 * A
    r = record([call("mmf_mlgru_fwd", A, 0, A, A, A, A, A, A, h, A, A, A, A, A, B, 1, 2048, A, BIG, None)])[0]
    assert r["status"] == 0 and kernels(r) == want
