"""K-split contraction of few token rows (skinny.hip) on the GPU.

Its int32 sums are exact and its epilogues evaluate the same expressions as the
tiled MFMA kernel's, so every output must equal the forced GEMM path's bit for
bit (that path is held to the oracle in test_gpu_parity.py, test_gpu_glu.py and
test_gpu_mlgru.py); the integer form is also checked against a plain int64
product here.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mmf():
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    import paper_2406_02528_amd as m
    return m


def both_paths(mmf, run):
    """run() on the automatic and on the forced GEMM path; outputs start as NaN."""
    out = []
    for path in (mmf.MMF_PATH_AUTO, mmf.MMF_PATH_GEMM):
        prev = mmf.mmf_set_path(path)
        try:
            out.append(run().cpu())
        finally:
            mmf.mmf_set_path(prev)
    return out


def nan(*shape):
    return torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")


def same(a, b):
    return a.shape == b.shape and not torch.isnan(a).any() and torch.equal(a, b)


def weights(mmf, N, K, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return mmf.ternarize(torch.randn(N, K, generator=g, device="cuda") * 0.02)


# The tile each shape runs on (256 compute units), as row blocks x column blocks
# / steps in flight, or the kernel that takes it instead; test_routes.py checks
# them without a GPU.  Together: every tile form, several row blocks with the
# last one partly filled or without whole blocks, ragged ends of the column
# strips, N odd and N % 4 == 2; K with a last step of 16, 32 and 48 features,
# fewer steps than waves, and more than two steps per wave.
FORWARD = {
    (17, 16, 100): "1x1/2", (17, 1040, 1000): "1x1/4", (31, 2064, 6000): "1x4/4", (33, 2096, 2044): "1x2/4",
    (45, 5632, 2048): "1x2/4", (47, 2080, 11266): "1x8/4", (64, 528, 301): "1x1/2", (65, 1024, 4096): "2x4/2",
    (70, 4112, 260): "1x1/4", (100, 2048, 11264): "2x8/2", (129, 1072, 3001): "2x4/4", (257, 2048, 1000): "1x4/4",
    (400, 112, 48): "1x1/2", (1, 16400, 96): "decode", (5, 13824, 324): "decode", (16, 13824, 5120): "1x2/4",
    (33, 1024, 5): "1x1/2",
    # the 64 x 256 tile (two column halves, four shares of K), ragged in each dimension
    (100, 2064, 27000): "4x16/2", (127, 1040, 27001): "4x16/2", (250, 4112, 15300): "4x16/2",
    # two and three row blocks (three: a last round of partial sums half
    # filled), tiles of a whole compute unit, at long K and ragged
    (39, 2096, 3298): "2x2/4", (97, 1616, 4589): "1x8/4", (153, 1040, 1872): "3x2/4", (150, 1040, 1873): "3x2/4",
    (128, 13824, 5120): "3x4/2", (128, 5120, 5120): "3x4/2", (93, 1040, 6864): "3x4/2", (115, 1040, 4649): "3x4/2",
    (130, 1664, 10380): "3x8/2", (84, 1040, 15358): "3x8/2", (112, 928, 13572): "4x8/2", (100, 1040, 15358): "4x8/2",
    (128, 5120, 15360): "4x8/2"}
RAW = {(17, 16, 100): "1x1/2", (45, 2096, 2044): "1x2/4", (100, 1040, 6001): "2x8/2", (130, 512, 8192): "2x8/2",
       (81, 1040, 6737): "3x4/2", (100, 144, 10865): "3x8/2", (50, 1040, 26221): "4x8/2", (437, 176, 1300): "3x4/2"}
GLU = {(17, 16, 16): "1x2/2", (33, 1040, 2832): "1x4/4", (45, 2048, 5632): "1x8/4", (200, 2064, 528): "1x4/4",
       (128, 5120, 1744): "2x4/4", (120, 1040, 13824): "tiled", (37, 1200, 1568): "2x2/4", (357, 2064, 720): "2x4/4",
       (183, 1184, 3888): "3x8/2", (196, 1120, 3744): "4x8/2", (130, 1312, 10272): "4x16/2", (308, 16, 816): "3x4/2"}
GATES = {(17, 64, 16): "1x1/2", (33, 1040, 1040): "2x2/4", (45, 2048, 2048): "2x4/4", (300, 528, 272): "1x4/2",
         (153, 1040, 624): "3x2/4", (128, 5120, 1712): "3x4/2", (325, 1264, 1536): "3x8/2", (298, 2800, 1984): "4x8/2",
         (74, 1392, 8608): "4x16/2"}


@pytest.mark.parametrize("M,K,N", FORWARD)
@pytest.mark.parametrize("f32", [False, True])
def test_forward_equals_the_gemm_path(mmf, M, K, N, f32):
    print(f"forward M={M} K={K} N={N} f32={f32}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn(M, K, generator=g, device="cuda")
    x = x if f32 else x.bfloat16()
    gamma = torch.rand(K, generator=g, device="cuda") + 0.5
    Wp, ws = weights(mmf, N, K, 8)
    w = torch.empty(mmf.mmf_bitlinear_workspace_bytes(M, K), dtype=torch.uint8, device="cuda")

    def run():
        y = nan(M, N)
        w.fill_(0x55)  # nothing may be read from the scratch before it is written
        mmf.mmf_bitlinear_fwd_ws(x, gamma, Wp, ws, y, w)
        return y
    a, b = both_paths(mmf, run)
    assert same(a, b)
    # the allocating form (up to 32 tokens decode launches, which need no scratch)
    assert torch.equal(mmf.bitlinear(x, gamma, Wp, ws).cpu(), b)


@pytest.mark.parametrize("M,K,N", RAW)
def test_integer_sums_from_rows_of_q(mmf, M, K, N):
    print(f"raw M={M} K={K} N={N}", flush=True)
    rs = np.random.default_rng(3)
    q = torch.from_numpy(rs.integers(-128, 128, (M, K), dtype=np.int8))
    W = torch.from_numpy(rs.standard_normal((N, K), dtype=np.float32) * np.float32(0.02))
    Wp, ws = mmf.ternarize(W.cuda())
    s = ws.cpu()
    t = torch.clamp(torch.round(W * (1.0 / s)), -1, 1).to(torch.int64)
    acc = torch.full((M, N), -7, dtype=torch.int32, device="cuda")
    mmf.mmf_ternary_gemm_i32(q.cuda(), Wp, acc)
    assert torch.equal(acc.cpu().to(torch.int64), q.to(torch.int64) @ t.t())


@pytest.mark.parametrize("M,K,L", GLU)
def test_glu_equals_the_gemm_path(mmf, M, K, L):
    print(f"glu M={M} K={K} L={L}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    (Wg, sg), (Wu, su) = weights(mmf, L, K, 1), weights(mmf, L, K, 2)
    Wgu, s2 = mmf.glu_pack(Wg, Wu), torch.cat([sg, su])
    w = torch.empty(mmf.mmf_bitlinear_workspace_bytes(M, K), dtype=torch.uint8, device="cuda")

    def run():
        p = nan(M, L)
        mmf.mmf_glu_fwd_ws(x, None, Wgu, s2, p, w)
        return p
    a, b = both_paths(mmf, run)
    assert same(a, b)


@pytest.mark.parametrize("M,K,d", GATES)
@pytest.mark.parametrize("full", [False, True])
def test_gates_equal_the_gemm_path(mmf, M, K, d, full):
    print(f"gates M={M} K={K} d={d} full={full}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(6)
    x = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    Wp, ws = weights(mmf, 3 * d, K, 4)
    s3 = torch.cat([ws, ws * 1.5, ws * 0.5])
    bias = torch.rand(3 * d, generator=g, device="cuda") - 0.5 if full else None
    lb = torch.rand(d, generator=g, device="cuda") if full else None
    w = torch.empty(mmf.mmf_mlgru_proj_workspace_bytes(M, K, d), dtype=torch.uint8, device="cuda")

    def run():
        o = nan(M, 3 * d)
        mmf.mmf_mlgru_proj(x, None, Wp, s3, bias, lb, o, w)
        return o
    a, b = both_paths(mmf, run)
    assert same(a, b)


@pytest.mark.parametrize("M", [20, 45])
def test_capture_and_replay(mmf, M):
    """Captured calls replay to the eager result, with caller scratch (K-split
    kernel) and without (the fused decode launches, which allocate nothing)."""
    K, N = 2048, 1000
    g = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    Wp, ws = weights(mmf, N, K, 8)
    w = torch.empty(mmf.mmf_bitlinear_workspace_bytes(M, K), dtype=torch.uint8, device="cuda")
    y, z = nan(M, N), nan(20, N)
    mmf.mmf_bitlinear_fwd_ws(x, None, Wp, ws, y, w)
    want = y.clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        mmf.mmf_bitlinear_fwd_ws(x, None, Wp, ws, y, w)
        mmf.mmf_bitlinear_fwd(x[:20], None, Wp, ws, z)
    for _ in range(3):
        y.fill_(float("nan"))
        z.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want) and torch.equal(z, want[:20])
