"""The kernels that calls of the C ABI launch (host side only: tests/record.py
records the launches of the built library on 256 compute units)."""
import pytest

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
