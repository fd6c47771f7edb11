"""The dense layer's bias through the staged stores of the tiled MFMA kernel,
the ternarisation's tiles, and the fixed-order sums of dW parts."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mmf():
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    import paper_2406_02528_amd as m
    return m


# one shape per tile form (64 x 256, 64 x 512, 128 x 512, paired 128 x 256),
# ragged in every dimension: y + bias added in fp32, bit for bit
@pytest.mark.parametrize("M,K,N", [(300, 1040, 2004), (1000, 336, 6004), (1100, 528, 8004), (3000, 400, 8204)])
def test_bias_equals_the_sum(mmf, M, K, N):
    print(f"bias M={M} K={K} N={N}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M)
    x = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    bias = torch.randn(N, generator=g, device="cuda")
    Wp, ws = mmf.ternarize(torch.randn(N, K, generator=g, device="cuda") * 0.02)
    prev = mmf.mmf_set_path(mmf.MMF_PATH_GEMM)
    try:
        y = mmf.bitlinear(x, None, Wp, ws)
        z = torch.full((M, N), float("nan"), device="cuda")
        mmf.mmf_bitlinear_fwd_bias(x, None, Wp, ws, bias, z)
    finally:
        mmf.mmf_set_path(prev)
    assert torch.equal(z, y + bias)


# tiles of 64 rows x 64 features: ragged rows, K with one to three words in its
# last tile, several blocks of the |W| sum
@pytest.mark.parametrize("N,K", [(1, 16), (63, 32), (65, 80), (1000, 112), (130, 1040), (2049, 2064)])
def test_ternarize_tiles(mmf, N, K):
    print(f"ternarize N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + K)
    W = torch.randn(N, K, generator=g, device="cuda") * 0.02
    Wp, ws = mmf.ternarize(W)
    mean = W.double().abs().mean().float().clamp_min(1e-5)
    assert abs(float(ws) - float(mean)) <= 1.2e-7 * float(mean)  # one fp32 ulp: fp64 sums in another order
    c = (torch.clamp(torch.round(W.cpu() * (1.0 / ws.cpu())), -1, 1).to(torch.int64) + 1).view(N, K // 16, 4, 4)
    i, b = torch.arange(4).view(1, 1, 4, 1), torch.arange(4).view(1, 1, 1, 4)
    words = (c << (8 * b + 2 * i)).sum((2, 3)).t()
    assert torch.equal(Wp.cpu().to(torch.int64) & 0xFFFFFFFF, words)
