"""Decoding (mla_recon_decode) at the edges of its kernels: sequence counts around the merge's
blocks of 8 and the query product's blocks of 32 rows, few and many key splits (the merge
takes them in two orders), empty splits and sequences, padded head counts, unaligned weights
and outputs; against a float64 evaluation of the same bf16 inputs."""
import pytest

from paper_2607_27269_amd import configs

pytestmark = pytest.mark.gpu
# bf16 roundings of the absorbed query, the probabilities, the latent and o, 2^-9 each in
# quadrature, 4e-3; the bound of the decoding parity tests
TOL = 1e-2


def _inputs(cfg, B, T, lengths, seed=3):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    rn = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).to(torch.bfloat16)
    H, dn, dr, rkv, dv, G = (cfg.n_heads, cfg.nope_dim, cfg.rope_dim, cfg.kv_rank, cfg.head_dim,
                             cfg.s_kv_groups)
    return dict(q=rn(B, H, dn + dr), cache=rn(B, T, rkv + dr), Wuk=rn(max(1, G * dn), rkv, std=rkv ** -0.5),
                Wuv=rn(G * dv, rkv, std=rkv ** -0.5),
                lens=torch.tensor(lengths, dtype=torch.int32, device="cuda"))


def _run(cfg, c, x, T, shift=0, ws=None):
    """shift: elements by which W_UK and o are moved off their 16-byte alignment; ws: the
    workspace (bytes), as its contents are."""
    import torch
    from paper_2607_27269_amd import _lib as L
    wsb = L.mla_recon_decode_workspace_size(c, T)
    assert wsb > 0, L.last_error()
    if ws is None:
        ws = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda")  # NaN patterns
    assert ws.numel() >= wsb
    n = cfg.batch * cfg.n_heads * cfg.head_dim
    ob = torch.full((n + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
    o = ob[shift:shift + n]
    wb = torch.empty(x["Wuk"].numel() + 8, dtype=torch.bfloat16, device="cuda")
    wuk = wb[shift:shift + x["Wuk"].numel()]
    wuk.copy_(x["Wuk"].reshape(-1))
    L.mla_recon_decode(c, x["q"].data_ptr(), x["cache"].data_ptr(), T, x["lens"].data_ptr(),
                       wuk.data_ptr(), x["Wuv"].data_ptr(), o.data_ptr(), ws.data_ptr(), wsb,
                       torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return o.reshape(cfg.batch, cfg.n_heads, cfg.head_dim)


def _reference(cfg, x, lengths):
    import torch
    q, cache, Wuk, Wuv = (x[n].double() for n in ("q", "cache", "Wuk", "Wuv"))
    G, dn, rkv, dv, H = cfg.s_kv_groups, cfg.nope_dim, cfg.kv_rank, cfg.head_dim, cfg.n_heads
    o = torch.zeros(cfg.batch, H, dv, dtype=torch.float64, device="cuda")
    for b, n in enumerate(lengths):
        if n == 0:
            continue
        c, pe = cache[b, :n, :rkv], cache[b, :n, rkv:]
        for i in range(H):
            g = i * G // H
            k = torch.cat([c @ Wuk[g * dn:(g + 1) * dn].T, pe], -1) if dn else pe
            o[b, i] = torch.softmax(k @ q[b, i] * cfg.softmax_scale, 0) @ (c @ Wuv[g * dv:(g + 1) * dv].T)
    return o


SMALL = dict(n_heads=6, n_kv_groups=2, s_kv_groups=2, hidden=384, kv_rank=128)


@pytest.mark.parametrize("idx,T,lengths,kw", [
    (3, 6000, [6000], {}),                                  # 47 splits: many to a slot
    (3, 2049, [2049, 1, 128, 129, 0, 2048, 700, 33, 5], {}),  # 17 splits, 9 sequences
    (3, 2048, [2048] * 7, {}),                              # 16 splits: the most of the other order
    (1, 5000, [5000, 3], {}), (1, 640, list(range(1, 641, 40)), {}),
    (2, 300, [300], {}), (2, 100, [100] * 33, {}),
    (2, 130, [130, 7], dict(nope_dim=0)),                   # no non-positional keys
    (1, 4500, [4500, 4499, 1], SMALL), (1, 200, [200] * 11, SMALL),
])
def test_decode_splits(idx, T, lengths, kw):
    import torch
    from paper_2607_27269_amd import _lib as L
    print(f"[splits] cfg{idx} T={T} B={len(lengths)} {kw}", flush=True)
    cfg = configs.get(idx).replace(batch=len(lengths), seq=T, **kw)
    c = L.make_cfg(cfg)
    x = _inputs(cfg, len(lengths), T, lengths)
    o = _run(cfg, c, x, T)
    ref = _reference(cfg, x, lengths)
    for b, n in enumerate(lengths):
        if n == 0:
            assert not o[b].float().any()
        else:
            e = float((o[b].double() - ref[b]).norm() / ref[b].norm())
            assert e <= TOL, (b, n, e)
    # neither W_UK nor o needs more alignment than its elements'
    assert torch.equal(o, _run(cfg, c, x, T, shift=3))


@pytest.mark.parametrize("idx,T,lengths,kw", [
    (1, 1500, [1500, 700, 1337], {}),    # 14 heads in a block of 32 columns
    (1, 4500, [4500, 4499, 1], SMALL),   # 6 heads
    (2, 900, [900, 450], dict(n_heads=40, hidden=2560)),  # 40 heads: the second block has 8
])
def test_decode_scratch_contents_do_not_change_results(idx, T, lengths, kw):
    """A head count that is no multiple of 32 leaves columns without a head; whatever the
    workspace held before (nothing, NaN patterns, finite values that grow from row to row, what
    another call left), the outputs are the same bits."""
    import torch
    from paper_2607_27269_amd import _lib as L
    B = len(lengths)
    cfg = configs.get(idx).replace(batch=B, seq=T, **kw)
    assert cfg.n_heads % 32
    c = L.make_cfg(cfg)
    x = _inputs(cfg, B, T, lengths)
    n = L.mla_recon_decode_workspace_size(c, T)
    assert n > 0, L.last_error()
    g = torch.Generator(device="cuda").manual_seed(9)
    ws = torch.zeros(n, dtype=torch.uint8, device="cuda")
    outs = {"zeros": _run(cfg, c, x, T, ws=ws)}
    outs["NaN patterns"] = _run(cfg, c, x, T, ws=ws.fill_(255))
    for scale in (1.0, 30.0, 1e4):
        # logits of a column in the order of scale: its maximum moves from key tile to key tile
        print(f"[scratch] cfg{idx} T={T} H={cfg.n_heads} scale {scale}", flush=True)
        row = cfg.kv_rank + cfg.rope_dim
        v = torch.randn(n // 2 // row + 1, row, device="cuda", generator=g)
        v *= scale * torch.linspace(0.5, 2, v.shape[0], device="cuda")[:, None]
        ws[:n // 2 * 2].view(torch.bfloat16).copy_(v.reshape(-1)[:n // 2])
        outs[f"finite, {scale}"] = _run(cfg, c, x, T, ws=ws)
    # what a call with more heads left: its absorbed queries lie where this call's columns
    # without a head are
    other = cfg.replace(n_heads=32 * ((cfg.n_heads + 31) // 32), n_kv_groups=2, s_kv_groups=2)
    co = L.make_cfg(other)
    xo = _inputs(other, B, T, [T] * B, seed=4)
    big = torch.zeros(L.mla_recon_decode_workspace_size(co, T), dtype=torch.uint8, device="cuda")
    _run(other, co, dict(xo, q=xo["q"] * 20), T, ws=big)
    outs["another call's"] = _run(cfg, c, x, T, ws=big)
    for k, o in outs.items():
        assert torch.equal(o, outs["zeros"]), k
