"""Output widths that are no multiple of 4 on the tiled MFMA kernel, and the
tile forms of the backward's dY kernel at their edges."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_train import mmf, run_bwd  # noqa: E402,F401


def codes(K, N, seed):
    """Random packed words: every code is 0, 1 or 2."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    lo = torch.randint(0, 1 << 32, (K // 16, N), generator=g, device="cuda", dtype=torch.int64) & 0x55555555
    hi = torch.randint(0, 1 << 32, (K // 16, N), generator=g, device="cuda", dtype=torch.int64) & 0x55555555
    return (lo + (hi & ~lo & 0x55555555) * 2).to(torch.int32)


# 64 x 256, 64 x 512, 128 x 512 and paired 128 x 256 tiles, each N % 4, ragged
# in every dimension, against the same columns of a matrix widened to a
# multiple of 4.
@pytest.mark.parametrize("M,K,N,plan", [(300, 1040, 2001, "64x256"), (1000, 336, 6002, "64x512"),
                                        (1100, 528, 8003, "128x512"), (3000, 400, 8201, "128x256_paired"),
                                        (257, 16, 5, "64x256")])
def test_odd_widths_equal_the_widened_matrix(mmf, M, K, N, plan):  # noqa: F811
    print(f"ragged M={M} K={K} N={N}", flush=True)
    assert mmf.mmf_prefill_tile_plan(M, K, N) == plan
    g = torch.Generator(device="cuda").manual_seed(N)
    q = torch.randint(-127, 128, (M, K), generator=g, device="cuda", dtype=torch.int8)
    rs = q.to(torch.int32).sum(1, dtype=torch.int32)
    a = torch.rand(M, generator=g, device="cuda") + 0.5
    ws = torch.tensor([0.02], device="cuda")
    wide = codes(K, (N + 3) // 4 * 4, 1)
    exact = wide[:, :N].contiguous()  # ends where the allocation's rows end
    prev = mmf.mmf_set_path(mmf.MMF_PATH_GEMM)
    try:
        want = torch.full((M, wide.shape[1]), float("nan"), device="cuda")
        mmf.mmf_ternary_gemm_dequant(q, a, rs, wide, ws, want)
        got = torch.full((M * N + 64,), -3.0, device="cuda")
        y = got[:M * N].view(M, N)
        y.fill_(float("nan"))
        mmf.mmf_ternary_gemm_dequant(q, a, rs, exact, ws, y)
        assert torch.equal(y, want[:, :N]) and (got[M * N:] == -3.0).all()
        acc_w = torch.full((M, wide.shape[1]), -7, dtype=torch.int32, device="cuda")
        acc = torch.full((M, N), -7, dtype=torch.int32, device="cuda")
        mmf.mmf_ternary_gemm_i32(q, wide, acc_w)
        mmf.mmf_ternary_gemm_i32(q, exact, acc)
        assert torch.equal(acc, acc_w[:, :N])
    finally:
        mmf.mmf_set_path(prev)


# dY on 64 x 256 and on 128 x 512 tiles (the tile of each on 256 compute units,
# checked without a GPU by test_routes.py), ragged in tokens and input
# features, N odd and N % 8 != 0 (dO rows on any 2 bytes, rows shorter than a
# chunk).
DY_TILES = {(65, 272, 9, False, True): (64, 256), (130, 1040, 127, True, True): (64, 256),
            (1937, 528, 77, False, False): (64, 256), (2, 16, 3, True, False): (64, 256),
            (16300, 1008, 40, False, True): (128, 512), (16300, 1008, 41, True, False): (128, 512)}


@pytest.mark.parametrize("M,K,N,f32_x,with_gamma", DY_TILES)
def test_dy_tiles(mmf, M, K, N, f32_x, with_gamma):  # noqa: F811
    print(f"dY M={M} K={K} N={N}", flush=True)
    run_bwd(mmf, M, K, N, f32_x, with_gamma, seed=11)


# More rows than pad_rows_kernel's grid: each workgroup then pads several.
def test_padding_of_very_many_rows(mmf):  # noqa: F811
    M, K, N = (1 << 22) + 9, 16, 3
    print(f"pad M={M} K={K} N={N}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    dO = torch.randn(M, N, generator=g, device="cuda").bfloat16()
    W = torch.randn(N, K, generator=g, device="cuda") * 0.02
    e = lambda *s, t=torch.float32: torch.empty(s, dtype=t, device="cuda")  # noqa: E731
    y, Wp, ws, q, a, r = e(M, N), e(1, N, t=torch.int32), e(1), e(M, K, t=torch.int8), e(M), e(M)
    mmf.mmf_bitlinear_train_fwd(x, None, W, None, y, Wp, ws, q, a, r)
    dx, dW, db = e(M, K).fill_(float("nan")), e(N, K), e(N)
    mmf.mmf_bitlinear_bwd(dO, x, None, r, q, a, Wp, ws, dx, dW, db, None)
    t = torch.clamp(torch.round(W.cpu() * (1.0 / ws.cpu())), -1, 1).double().cuda()
    xd, rd = x.double(), r.double()[:, None]
    def parts(d, t, x):  # the two terms of dx
        dY = (d @ t) * ws.double()
        return rd * dY, x * (dY * x).sum(1, keepdim=True) * rd ** 3 / K

    p1, p2 = parts(dO.double(), t, xd)
    # fp32: a sum of three exact products (rounded relative to the sum of their
    # magnitudes), its factors and the difference, fewer than 16 roundings of
    # 2^-24: 1e-6 of the terms formed from magnitudes
    b1, b2 = parts(dO.double().abs(), t.abs(), xd.abs())
    assert ((dx.double() - (p1 - p2)).abs() <= 1e-6 * (b1 + b2)).all()
    ref = dO.double().sum(0)  # fp64 on both sides, rounded once: 2^-24, and 2^-52 per addend
    assert ((db.double() - ref).abs() <= 1e-7 * ref.abs() + 1e-15 * dO.double().abs().sum(0)).all()
