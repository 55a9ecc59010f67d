"""Token counts at the edges of the products' and the attention's tiles (64, 128, 192 and 256
rows, 32-query blocks, 256-key blocks): the whole step against the float64 oracle, so that
every projection, data gradient and weight gradient runs with a tile that the matrix edge
cuts, with a matrix smaller than a tile, and with a ragged reduction length."""
import numpy as np
import pytest

from paper_2607_27269_amd import configs, synth
from parity_util import LOSS_TOL, TOL, compare, oracle_step

pytestmark = pytest.mark.gpu

GRADS = ("dWdq", "dWuq", "dWdkv_kr", "dWuk", "dWuv")


# The gradients carry the relative error of A_s - A_t: sqrt(2) * 3.2e-3 (the bf16 error of each
# output) times |A_t| / |A_s - A_t|, which is 2.5 for 63 tokens of configuration 1 (dA alone
# 1.2e-2, its dW_UV 1.9e-2 and a group of it 2.2e-2) and nears 1 for longer sequences.  A
# gradient sums products with it, whose own sum can cancel: twice that, and twice for margin.
# A tile gone wrong shows as 1e-1 and more in its block.
DA_ERR = 2 ** 0.5 * 3.2e-3


def _tol(wl, ref):
    m = wl.mask[..., None]
    return max(TOL["bf16"], 4 * DA_ERR * np.linalg.norm(m * ref["A_t"]) /
               np.linalg.norm(m * (ref["A_s"] - ref["A_t"])))


@pytest.mark.parametrize("idx,B,T", [(4, 1, 33), (1, 1, 63), (1, 2, 65), (1, 1, 129), (1, 3, 85),
                                     (1, 1, 257), (2, 1, 191), (2, 1, 321), (4, 1, 96), (2, 4, 1021),
                                     (2, 7, 883)])
def test_step_sizes(idx, B, T):
    from paper_2607_27269_amd.step import DeviceStep
    print(f"[sizes] cfg{idx} B={B} T={T}", flush=True)
    cfg = configs.shrink(configs.get(idx), batch=B, seq=T)
    wl = synth.make_workload(cfg, lengths=[T] * (B - 1) + [max(1, T - 5)])
    ref = oracle_step(wl)
    tol = _tol(wl, ref)
    dev = DeviceStep(wl)
    dev.step()
    out = dev.results()
    compare(out, ref, ("A_t", "A_s"), TOL["bf16"], label="four calls: ", cfg=cfg)
    compare(out, ref, ("dA",) + GRADS, tol, label="four calls: ", cfg=cfg)
    assert abs(out["loss"] - ref["loss"]) <= LOSS_TOL * ref["loss"]
    for with_dA in (False, True):
        for g in dev.grads.values():
            g.fill_(float("nan"))
        dev.fused_step(with_dA=with_dA)
        out = dev.results()
        compare(out, ref, GRADS, tol, label=f"single call, dA={with_dA}: ", cfg=cfg)
        assert abs(out["loss"] - ref["loss"]) <= LOSS_TOL * ref["loss"]


@pytest.mark.parametrize("dv,dn,dr,Gr,B,T", [(32, 32, 32, 1, 2, 200), (32, 16, 16, 2, 1, 130),
                                             (16, 8, 8, 2, 3, 77)])
def test_step_narrow_heads_bf16(dv, dn, dr, Gr, B, T):
    """Head widths that only the vector-ALU attention has, in bf16 (its dQ is summed in an
    fp32 region of its own)."""
    from paper_2607_27269_amd.step import DeviceStep
    print(f"[sizes] d_k={dv} d_nope={dn} d_rope={dr} B={B} T={T}", flush=True)
    cfg = configs.shrink(configs.get(1), batch=B, seq=T, hidden=512, n_heads=8, n_kv_groups=2, head_dim=dv,
                         q_rank=128, kv_rank=64, nope_dim=dn, rope_dim=dr, s_kv_groups=2, s_rope_groups=Gr,
                         outlier_channels=0)
    wl = synth.make_workload(cfg)
    ref = oracle_step(wl)
    tol = _tol(wl, ref)
    dev = DeviceStep(wl)
    for label, step in (("four calls: ", dev.step), ("single call: ", lambda: dev.fused_step(with_dA=False))):
        for g in dev.grads.values():
            g.fill_(float("nan"))
        dev.ws.fill_(255)  # NaN patterns
        step()
        out = dev.results()
        compare(out, ref, [g for g in GRADS if g in dev.grads], tol, label=label, cfg=cfg)
        assert abs(out["loss"] - ref["loss"]) <= LOSS_TOL * ref["loss"]


@pytest.mark.parametrize("B,T", [(2, 640), (3, 130), (5, 333)])
def test_step_workspace_does_not_change_results(B, T):
    """Neither the split of a product nor that of a group's heads (and with them the rounding)
    depends on how much workspace the caller gives: the backward in chunks of one sequence, in
    even and uneven chunks and in one pass gives the same bits."""
    import torch
    from paper_2607_27269_amd import _lib as L
    from paper_2607_27269_amd.step import DeviceStep
    cfg = configs.shrink(configs.get(1), batch=B, seq=T)
    wl = synth.make_workload(cfg)
    c = L.make_cfg(cfg)
    lo, hi = L.mla_recon_workspace_size_min(c), L.mla_recon_workspace_size(c)
    assert hi - lo > (B - 1) * 2 * T * T * cfg.n_heads  # a sequence's dS^T each
    # chunks of 1 .. B sequences: one more for each equal part between the two sizes
    sizes = [hi] + [lo + (hi - lo) * n // (B - 1) + 4096 for n in range(B - 1)]
    outs = []
    for ws_bytes in sizes:
        print(f"[workspace] B={B} T={T} {ws_bytes}", flush=True)
        dev = DeviceStep(wl, ws_bytes=ws_bytes)
        dev.ws.fill_(255)  # NaN patterns
        dev.fused_step(with_dA=False)
        torch.cuda.synchronize()
        outs.append({"loss": dev.loss_buf[:1].clone(), **{k: v.clone() for k, v in dev.grads.items()}})
    for o in outs[1:]:
        for k in outs[0]:
            assert torch.equal(outs[0][k], o[k]), k
    assert all(torch.isfinite(v).all() for v in outs[0].values())
