"""Prefill (mla_recon_prefill) at the edges of its attention tiles (32-query wavefronts,
64-key tiles, 256-query workgroups) in every output form, against a float64 evaluation of
the same bf16 inputs, and its treatment of non-finite cache rows."""
import numpy as np
import pytest

from paper_2607_27269_amd import configs

pytestmark = pytest.mark.gpu
# o and A carry the bf16 roundings of the keys, values (or latents), probabilities and o:
# about four of 2^-9 each, added in quadrature, 4e-3; the bound of the decoding tests
TOL = 1e-2


def _setup(idx, B, T, seed=5, **kw):
    import torch
    from paper_2607_27269_amd import _lib as L
    cfg = configs.get(idx).replace(batch=B, seq=T, **kw)
    g = torch.Generator(device="cuda").manual_seed(seed)
    rn = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).to(torch.bfloat16)
    H, dn, dr, rkv, dv, G = (cfg.n_heads, cfg.nope_dim, cfg.rope_dim, cfg.kv_rank, cfg.head_dim,
                             cfg.s_kv_groups)
    x = dict(q=rn(B, T, H, dn + dr), cache=rn(B, T, rkv + dr), Wuk=rn(max(G * dn, 1), rkv, std=rkv ** -0.5),
             Wuv=rn(G * dv, rkv, std=rkv ** -0.5), Wo=rn(cfg.hidden, H * dv, std=(H * dv) ** -0.5))
    c = L.make_cfg(cfg)
    wsb = L.mla_recon_prefill_workspace_size(c)
    assert wsb > 0, L.last_error()
    x["ws"] = torch.full((wsb,), 255, dtype=torch.uint8, device="cuda")  # NaN patterns
    x["fold"] = torch.empty(cfg.hidden, H * rkv, dtype=torch.bfloat16, device="cuda")
    L.mla_recon_fold_uv_into_o(c, x["Wo"].data_ptr(), x["Wuv"].data_ptr(), x["fold"].data_ptr(),
                               torch.cuda.current_stream().cuda_stream)
    return cfg, c, x


def _run(cfg, c, x, form, o_shift=0):
    import torch
    from paper_2607_27269_amd import _lib as L
    n = cfg.batch * cfg.seq * cfg.n_heads * cfg.head_dim
    want_o, want_a, folded = form in ("o", "o+A", "o+folded"), form != "o", "folded" in form
    ob = torch.full((n + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
    o = ob[o_shift:o_shift + n]
    A = torch.full((cfg.batch * cfg.seq, cfg.hidden), float("nan"), device="cuda")
    p = lambda t, on: t.data_ptr() if on else None
    L.mla_recon_prefill(c, x["q"].data_ptr(), x["cache"].data_ptr(), x["Wuk"].data_ptr(),
                        p(x["Wuv"], want_o or not folded), p(x["Wo"], not folded), p(x["fold"], folded),
                        p(o, want_o), p(A, want_a), x["ws"].data_ptr(), x["ws"].numel(),
                        torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    o = o.reshape(cfg.batch, cfg.seq, cfg.n_heads, cfg.head_dim)
    return o if want_o else None, A.reshape(cfg.batch, cfg.seq, -1) if want_a else None


def _reference(cfg, x):
    import torch
    q, cache, Wuk, Wuv, Wo = (x[n].double() for n in ("q", "cache", "Wuk", "Wuv", "Wo"))
    G, dn, rkv, dv, H, T = (cfg.s_kv_groups, cfg.nope_dim, cfg.kv_rank, cfg.head_dim, cfg.n_heads, cfg.seq)
    o = torch.zeros(cfg.batch, T, H, dv, dtype=torch.float64, device="cuda")
    future = torch.ones(T, T, dtype=torch.bool, device="cuda").triu_(1)
    for b in range(cfg.batch):
        c, pe = cache[b, :, :rkv], cache[b, :, rkv:]
        for i in range(H):
            g = i * G // H
            k = torch.cat([c @ Wuk[g * dn:(g + 1) * dn].T, pe], -1) if dn else pe
            S = (q[b, :, i] @ k.T * cfg.softmax_scale).masked_fill(future, float("-inf"))
            o[b, :, i] = torch.softmax(S, -1) @ (c @ Wuv[g * dv:(g + 1) * dv].T)
    return o, o.reshape(cfg.batch, T, -1) @ Wo.T


def _rel(x, ref):
    return float((x.double() - ref).norm() / ref.norm())


@pytest.mark.parametrize("idx,B,T,form,kw", [
    (3, 1, 1, "o+A", {}), (3, 2, 65, "o+folded", {}), (3, 1, 257, "folded", {}),
    (1, 3, 33, "A", {}), (1, 1, 256, "o+A", {}), (1, 2, 511, "folded", {}),
    (2, 1, 63, "o", {}), (2, 2, 97, "o+folded", {}),
    # no non-positional keys; odd head count per group; rank 128
    (2, 2, 70, "o+A", dict(nope_dim=0)), (2, 1, 40, "folded", dict(nope_dim=0)),
    (1, 2, 129, "o+folded", dict(n_heads=6, n_kv_groups=2, s_kv_groups=2, hidden=384, kv_rank=128)),
])
def test_prefill_forms(idx, B, T, form, kw):
    print(f"[prefill] cfg{idx} B={B} T={T} {form} {kw}", flush=True)
    cfg, c, x = _setup(idx, B, T, **kw)
    o, A = _run(cfg, c, x, form)
    o_ref, A_ref = _reference(cfg, x)
    if o is not None:
        assert _rel(o, o_ref) <= TOL
        for t in sorted({0, T - 1, T // 2, min(31, T - 1), min(32, T - 1)}):
            assert _rel(o[:, t], o_ref[:, t]) <= 2 * TOL
    if A is not None:
        assert _rel(A, A_ref) <= TOL


def test_prefill_unaligned_o():
    """o needs no alignment beyond its elements': the same values as the aligned call."""
    import torch
    cfg, c, x = _setup(1, 2, 50)
    for form in ("o+A", "o+folded"):
        o, A = _run(cfg, c, x, form)
        o1, A1 = _run(cfg, c, x, form, o_shift=3)
        assert torch.equal(o, o1) and torch.equal(A, A1)


def test_prefill_unaligned_weights():
    """A prefill of few tokens takes W_UK and W_O (or W_O') at any element: the same bits."""
    import torch
    cfg, c, x = _setup(1, 2, 30)
    for form in ("o+A", "o+folded"):
        o, A = _run(cfg, c, x, form)
        for shift in (1, 2, 4):
            y = dict(x)
            for n in ("Wuk", "Wo", "fold"):
                b = torch.empty(x[n].numel() + 8, dtype=x[n].dtype, device="cuda")
                y[n] = b[shift:shift + x[n].numel()]
                y[n].copy_(x[n].reshape(-1))
            print(f"[prefill] {form} weights moved by {shift}", flush=True)
            o1, A1 = _run(cfg, c, y, form)
            assert torch.equal(o, o1) and torch.equal(A, A1)


@pytest.mark.parametrize("idx,form", [(1, "o+A"), (1, "folded"), (3, "o+A"), (2, "o+folded")])
@pytest.mark.parametrize("row", [0, 37, 66, 99])
def test_prefill_nonfinite_rows(idx, form, row):
    """A cache row with a NaN or an infinity: NaN for the tokens that see it (row 0 of the
    last sequence: all of that one), the outputs of all other tokens bitwise unchanged."""
    import torch
    B, T = 2, 100
    cfg, c, x = _setup(idx, B, T)
    o, A = _run(cfg, c, x, form)
    for bad in (float("nan"), float("inf"), float("-inf")):
        print(f"[prefill] cfg{idx} {form} row {row} {bad}", flush=True)
        x2 = dict(x, cache=x["cache"].clone())
        x2["cache"][1, row, 5] = bad
        o2, A2 = _run(cfg, c, x2, form)
        for y, y2 in ((o, o2), (A, A2)):
            if y is None:
                continue
            assert torch.equal(y[0], y2[0]) and torch.equal(y[1, :row], y2[1, :row])
            assert not torch.isfinite(y2[1, row:].float()).any()


@pytest.mark.parametrize("idx,form", [(1, "o+A"), (3, "A"), (2, "o+folded"), (1, "folded")])
def test_prefill_huge_finite_rows(idx, form):
    """Cache rows past the tokens in use may hold any finite bytes, whose values W_UV c lie
    beyond bf16: the tokens before them are as with zeros there.  (Not bitwise: the softmax
    reference of a wavefront's queries moves together.)"""
    import torch
    B, T, n = 2, 200, 70
    cfg, c, x = _setup(idx, B, T)
    x["cache"][:, n:] = 0
    o, A = _run(cfg, c, x, form)
    g = torch.Generator(device="cuda").manual_seed(6)
    sign = torch.randint(0, 2, x["cache"][:, n:].shape, device="cuda", generator=g) * 2 - 1
    for big in (3e38, 2.0 ** 70):
        print(f"[prefill] cfg{idx} {form} rows of {big}", flush=True)
        x2 = dict(x, cache=x["cache"].clone(), Wuv=x["Wuv"] * (1.0 if big > 1e38 else 2.0 ** 57))
        x2["cache"][:, n:] = (sign * big).to(torch.bfloat16)
        x1 = dict(x, Wuv=x2["Wuv"])
        y1 = (o, A) if big > 1e38 else _run(cfg, c, x1, form)
        for y, y2 in zip(y1, _run(cfg, c, x2, form)):
            if y is not None:
                assert torch.isfinite(y2[:, :n].float()).all()
                assert _rel(y2[:, :n], y[:, :n].double()) <= TOL
