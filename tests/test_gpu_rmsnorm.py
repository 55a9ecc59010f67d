"""The residual add and RMS normalisation at the edges of its vector kernel (row widths around
1024, 2048, 4096 and 8192 values, widths that are not multiples of four, unaligned arrays)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("D,shift", [(1, 0), (3, 0), (4, 0), (1020, 0), (1024, 0), (1028, 0), (2048, 0),
                                     (2052, 0), (4096, 0), (4096, 1), (4100, 0), (8192, 0), (8196, 0)])
def test_residual_rmsnorm_widths(D, shift, dtype):
    import torch
    from paper_2607_27269_amd import _lib as L
    N, eps = 5, 1e-6
    g = torch.Generator(device="cuda").manual_seed(D)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    new = lambda: torch.randn(N * D + shift, device="cuda", generator=g)[shift:]
    x0, A = new(), new()
    for with_A in (True, False):
        x = torch.empty(N * D + shift, device="cuda")[shift:]
        x.copy_(x0)
        h = torch.full((N * D + shift,), float("nan"), device="cuda", dtype=tdt)[shift:]
        L.mla_recon_residual_rmsnorm(x.data_ptr(), A.data_ptr() if with_A else None, h.data_ptr(), N, D,
                                     L.MLA_FP32 if dtype == "fp32" else L.MLA_BF16, eps,
                                     torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        want = x0 + A if with_A else x0
        assert torch.equal(x, want)  # the fp32 add is exact to the bit
        w = want.double().reshape(N, D)
        ref = w * torch.rsqrt(w.square().mean(-1, keepdim=True) + eps)
        # fp32: a sum of D squares in any order is within D 2^-24 of exact at worst, and
        # within a few 2^-24 as summed here; bf16: half a unit in the last place, 2^-9
        tol = 2.0 ** -8 if dtype == "bf16" else 1e-6
        assert float(((h.double().reshape(N, D) - ref).abs() / ref.abs().clamp_min(1e-3)).max()) <= tol
