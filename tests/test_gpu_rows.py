"""Activation rows: the wave counts of act-quant (one to sixteen waves per
row, and rows past its registers), and the MLGRU decode step inside it, which
must give the bits of the separate kernels."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import workloads  # noqa: E402
from _parity import compare_q, to_dev_x  # noqa: E402


@pytest.fixture(scope="module")
def mmf():
    if not torch.cuda.is_available():
        pytest.skip("needs a HIP device")
    import paper_2406_02528_amd as m
    return m


# 45 rows: several waves for rows that one would hold; fp32 8208 .. 32768 and
# bf16 16400 .. 65536 on 8 and 16 waves, beyond that re-read from memory.
@pytest.mark.parametrize("M,K,f32", [(45, 2048, False), (45, 2048, True), (65, 2048, False), (3, 8208, True),
                                     (2, 16400, True), (1, 32768, True), (2, 32784, True), (3, 16400, False),
                                     (1, 65536, False), (2, 65552, False), (130, 13824, True)])
def test_act_quant_rows(mmf, M, K, f32):
    print(f"act_quant M={M} K={K} f32={f32}", flush=True)
    rs = np.random.default_rng(K + M)
    x = (rs.standard_normal((M, K)) * rs.uniform(0.1, 10.0, (M, 1))).astype(np.float32)
    bits = workloads.f32_to_bf16_bits(x)
    xf = x if f32 else workloads.bf16_bits_to_f32(bits)
    gamma = rs.uniform(0.5, 1.5, K).astype(np.float32)
    q = torch.full((M, K), 99, dtype=torch.int8, device="cuda")
    a = torch.full((M,), float("nan"), device="cuda")
    s = torch.full((M,), -1, dtype=torch.int32, device="cuda")
    mmf.mmf_act_quant(to_dev_x(x if f32 else bits), torch.from_numpy(gamma).cuda(), q, a, s)
    q_ref, a_ref = oracle.rmsnorm_act_quant(xf, gamma)
    compare_q(q.cpu().numpy(), q_ref)
    assert np.abs(a.cpu().numpy() - a_ref).max() <= 1e-6 * np.abs(a_ref).max()
    assert np.array_equal(s.cpu().numpy(), q.cpu().numpy().astype(np.int32).sum(1))


@pytest.mark.parametrize("B,d", [(17, 48), (45, 2048), (100, 1040), (3, 5120), (1, 5120), (2, 16400)])
@pytest.mark.parametrize("state", ["none", "apart", "in place"])
def test_decode_step_equals_its_stages(mmf, B, d, state):
    """One token of each sequence through the mixer against the projection, the
    recurrence kernel and the biased dense layer as three calls."""
    print(f"step B={B} d={d} state={state}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(B + d)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    x, gamma, gamma_o = r(B, d).bfloat16(), r(d).abs() + 0.5, r(d).abs() + 0.5
    words = lambda n: torch.randint(0, 1 << 30, (d // 16, n), generator=g, device="cuda", dtype=torch.int32) & 0x15555555  # noqa: E731
    Wf, Wo = words(3 * d), words(d)
    s3, so = r(3).abs() * 0.02, r(1).abs() * 0.02
    bias, lb, b_o = r(3 * d) * 0.3, torch.rand(d, generator=g, device="cuda"), r(d)
    h0 = None if state == "none" else r(B, d)
    fcg = mmf.mlgru_proj(x, gamma, Wf, s3, bias, lb)
    op, h_ref = mmf.mlgru_scan(fcg, B, 1, h0)
    o_ref = torch.full((B, d), float("nan"), device="cuda")
    mmf.mmf_bitlinear_fwd_bias(op, gamma_o, Wo, so, b_o, o_ref)
    h = h0.clone() if state == "in place" else torch.full((B, d), float("nan"), device="cuda")
    h_in = h if state == "in place" else h0
    o = torch.full((B, d), float("nan"), device="cuda")
    ws = torch.empty(mmf.mmf_mlgru_workspace_bytes(B, 1, d), dtype=torch.uint8, device="cuda").fill_(0x55)
    mmf.mmf_mlgru_fwd(x, B, 1, gamma, Wf, s3, bias, lb, h_in, h, gamma_o, Wo, so, b_o, o, ws)
    assert torch.equal(h, h_ref) and torch.equal(o, o_ref)


# One token whose fp32 row takes all 16 waves of the fused decode kernel (two
# and four vectors per lane, partly filled), on either side of its range.
@pytest.mark.parametrize("K,N", [(4096, 100), (4112, 100), (5632, 2048), (8192, 301), (8208, 64), (13824, 5120),
                                 (16384, 40), (16400, 40)])
def test_one_token_with_a_long_row(mmf, K, N):
    print(f"long row K={K} N={N}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(K)
    x = torch.randn(1, K, generator=g, device="cuda")
    gamma = torch.rand(K, generator=g, device="cuda") + 0.5
    Wp, ws = mmf.ternarize(torch.randn(N, K, generator=g, device="cuda") * 0.02)
    q = torch.empty((1, K), dtype=torch.int8, device="cuda")
    a, s = torch.empty(1, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda")
    mmf.mmf_act_quant(x, gamma, q, a, s)
    want = torch.full((1, N), float("nan"), device="cuda")
    mmf.mmf_ternary_gemm_dequant(q, a, s, Wp, ws, want)
    assert torch.equal(mmf.bitlinear(x, gamma, Wp, ws), want)
    if N % 32 == 0:
        glu, ref = mmf.glu(x, gamma, Wp, torch.cat([ws, ws])), torch.full((1, N // 2), float("nan"), device="cuda")
        mmf.mmf_ternary_gemm_glu(q, a, s, Wp, torch.cat([ws, ws]), ref)
        assert torch.equal(glu, ref)
