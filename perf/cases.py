"""Workloads by which the library's speed is judged, each through its public entry points.

The calls are those a user of the library makes: the reconstruction step in one call and in
four, a training iteration on a cached teacher (student step, then AdamW), one layer of
calibration capture, decoding with and without a workspace, and causal prefill.  Layer
shapes are the repository's configurations 1-4; tokens, sequences, masks and cache lengths
span small and ragged calls up to the full sizes.

``listed`` names the fixed cases, ``draw`` makes more of the same ranges, ``prepare`` builds
what a program holds before the call, ``run`` is one pass, ``work`` its least bytes and
operations, ``tolerance`` the difference two correct bf16 implementations show, ``exact``
the same outputs in float64 by plain torch.
"""
from __future__ import annotations

import math

import torch

from paper_2607_27269_amd import _lib as L
from paper_2607_27269_amd import configs

DEV = "cuda:0"
BF = torch.bfloat16
GRADS = ("dWdq", "dWuq", "dWdkv_kr", "dWuk", "dWuv")
OPT = dict(lr=1e-5, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01)
OPT_STEP0 = 200  # the optimizer is mid-training: moments are non-zero, bias corrections small


# ---- the cases ---------------------------------------------------------------------------
def listed():
    return [
        # the benchmark's layer at its full calibration minibatch: the training step
        dict(name="step-8b-4x4096", kind="step", config=3, batch=4, seq=4096, padded=False),
        # the multi-head teacher with per-head positional keys, sequences of a ragged length
        dict(name="step-mha-2x3001", kind="step", config=4, batch=2, seq=3001, padded=False),
        # a 1B draft model's layer at its full minibatch, right-padded sequences
        dict(name="step-1b-8x2048-pad", kind="step", config=2, batch=8, seq=2048, padded=True),
        # a small minibatch of the smallest draft model, odd length
        dict(name="step-05b-3x777-pad", kind="step", config=1, batch=3, seq=777, padded=True),
        # the step in four calls, every intermediate returned: a debugging / logging run
        dict(name="fourcall-1b-2x333", kind="fourcall", config=2, batch=2, seq=333, padded=True),
        # a training iteration of the minibatch loop: cached teacher, student step, AdamW
        dict(name="train-05b-8x2048", kind="train", config=1, batch=8, seq=2048, padded=False),
        # calibration capture of one frozen layer: teacher, residual add, RMS norm
        dict(name="capture-8b-2x4096", kind="capture", config=3, batch=2, seq=4096),
        # serving: one token for each of 64 sequences over full caches (the benchmark's decode)
        dict(name="decode-8b-64x4096", kind="decode", config=3, batch=64, seq=4096, ragged=False,
             noalloc=False),
        # serving one user: a single sequence, latency counts
        dict(name="decode-8b-1x6000", kind="decode", config=3, batch=1, seq=6000, ragged=False,
             noalloc=True),
        # speculative drafting with the small model: a few sequences of mixed lengths
        dict(name="decode-05b-13x1500", kind="decode", config=1, batch=13, seq=1500, ragged=True,
             noalloc=True),
        # prompts entering the cache: per-head outputs and the block's output
        dict(name="prefill-8b-2x2048", kind="prefill", config=3, batch=2, seq=2048, form="o+A"),
        # the same for the small model with W_UV folded into W_O, odd length
        dict(name="prefill-05b-3x999-fold", kind="prefill", config=1, batch=3, seq=999,
             form="folded"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "step", "fourcall", "train", "capture", "decode", "decode",
                       "prefill", "prefill"))
    if kind in ("step", "fourcall", "train"):
        config = rng.randint(1, 4)
        full = configs.get(config)
        seq = _log_int(rng, 64, full.seq)
        if rng.random() < 0.4:
            seq = min(full.seq, max(64, seq // 64 * 64))
        batch = rng.randint(1, max(1, min(8, full.tokens // seq)))
        return dict(kind=kind, config=config, batch=batch, seq=seq, padded=rng.random() < 0.5)
    if kind == "capture":
        config = rng.randint(1, 4)
        seq = _log_int(rng, 64, 4096)
        return dict(kind=kind, config=config, batch=rng.randint(1, max(1, min(8, 8192 // seq))),
                    seq=seq)
    if kind == "decode":
        seq = _log_int(rng, 64, 16384)
        batch = _log_int(rng, 1, max(1, min(96, 64 * 4096 // seq)))
        return dict(kind=kind, config=rng.randint(1, 3), batch=batch, seq=seq,
                    ragged=rng.random() < 0.5, noalloc=batch <= 24 and rng.random() < 0.5)
    seq = _log_int(rng, 64, 2048)
    batch = rng.randint(1, max(1, min(8, 4096 // seq)))
    return dict(kind=kind, config=rng.randint(1, 3), batch=batch, seq=seq,
                form=rng.choice(("o", "A", "o+A", "folded")))


def _cfg(case):
    return configs.get(case["config"]).replace(batch=case["batch"], seq=case["seq"])


# ---- inputs ------------------------------------------------------------------------------
class _Draw:
    """Seeded Gaussian tensors on the GPU, in a fixed order."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV).manual_seed(seed)

    def __call__(self, *shape, std=1.0):
        return torch.randn(*shape, device=DEV, generator=self.g, dtype=torch.float32) * std

    def ints(self, lo, hi, n):
        return torch.randint(lo, hi + 1, (n,), device=DEV, generator=self.g)


def _hidden(cfg, rnd):
    """RMS-normalised tokens with a few outlier channels, bf16 [B*T, D]."""
    h = rnd(cfg.tokens, cfg.hidden)
    if cfg.outlier_channels:
        h[:, : cfg.outlier_channels] *= cfg.outlier_scale
    return (h * torch.rsqrt(h.square().mean(-1, keepdim=True) + 1e-6)).to(BF)


def _mask(cfg, rnd, padded):
    if not padded:
        return torch.ones(cfg.tokens, dtype=torch.uint8, device=DEV)
    valid = rnd.ints(max(1, cfg.seq // 2), cfg.seq, cfg.batch)
    t = torch.arange(cfg.seq, device=DEV)
    return (t[None, :] < valid[:, None]).to(torch.uint8).reshape(-1).contiguous()


def _teacher(cfg, rnd):
    D, dk = cfg.hidden, cfg.head_dim
    w = dict(Wq=rnd(cfg.n_heads * dk, D, std=D ** -0.5), Wk=rnd(cfg.n_kv_groups * dk, D, std=D ** -0.5),
             Wv=rnd(cfg.n_kv_groups * dk, D, std=D ** -0.5),
             Wo=rnd(D, cfg.n_heads * dk, std=(cfg.n_heads * dk) ** -0.5))
    p = torch.arange(dk // 2, device=DEV, dtype=torch.float64)
    inv = (cfg.rope_theta ** (-2.0 * p / dk)).float()
    return {k: v.to(BF) for k, v in w.items()}, inv


def _student(cfg, rnd, tw, inv):
    """A converted block of the teacher: keys, values and queries through a random
    low-rank subspace of the hidden space, positional rows of the group-mean key."""
    D, G, dk, dn, dr, Gr = (cfg.hidden, cfg.n_kv_groups, cfg.head_dim, cfg.nope_dim, cfg.rope_dim,
                            cfg.s_rope_groups)
    half, nr = dk // 2, dr // 2
    Wk = tw["Wk"].float().view(G, dk, D)
    Wq = tw["Wq"].float().view(cfg.n_heads, dk, D)
    keep = torch.arange(nr, device=DEV)  # rotary pairs kept by the positional key
    rows = torch.cat([keep, keep + half])
    drop = torch.ones(dk, dtype=torch.bool, device=DEV)
    drop[rows] = False
    shared = Gr < G
    if shared:
        Wkr = Wk[:, rows].mean(0)
        knope = Wk.clone()
        knope[:, rows] -= Wkr
        qnope = Wq
    else:
        Wkr = Wk[:, rows].reshape(Gr * dr, D)
        knope, qnope = Wk[:, drop], Wq[:, drop]
    P = rnd(cfg.kv_rank, D, std=D ** -0.5)
    q = torch.cat([qnope, Wq[:, rows]], dim=1).reshape(-1, D)
    w = dict(Wdq=None, Wuq=q)
    if cfg.q_rank:
        Pq = rnd(cfg.q_rank, D, std=D ** -0.5)
        w = dict(Wdq=Pq, Wuq=q @ Pq.T)
    w["Wdkv_kr"] = torch.cat([P, Wkr], dim=0)
    w["Wuk"] = knope.reshape(-1, D) @ P.T
    w["Wuv"] = tw["Wv"].float() @ P.T
    w = {k: None if v is None else (v + rnd(*v.shape, std=1e-3)).to(BF).contiguous()
         for k, v in w.items()}
    return w, inv[keep].repeat(Gr, 1).contiguous()


def _layer(case, seed):
    cfg = _cfg(case)
    rnd = _Draw(seed)
    x = dict(cfg=cfg, h=_hidden(cfg, rnd), mask=_mask(cfg, rnd, case.get("padded", False)))
    x["tw"], x["inv_t"] = _teacher(cfg, rnd)
    x["sw"], x["inv_s"] = _student(cfg, rnd, x["tw"], x["inv_t"])
    if case["kind"] == "train":
        x["m"] = {n: rnd(*x["sw"]["W" + n[2:]].shape, std=3e-6) for n in GRADS
                  if x["sw"]["W" + n[2:]] is not None}
        x["v"] = {n: rnd(*m.shape, std=1e-5).square() + 1e-11 for n, m in x["m"].items()}
    return x


def _capture(case, seed):
    cfg = _cfg(case)
    rnd = _Draw(seed)
    x = dict(cfg=cfg, h=_hidden(cfg, rnd), x=rnd(cfg.tokens, cfg.hidden))
    x["tw"], x["inv_t"] = _teacher(cfg, rnd)
    return x


def _attend(case, seed):
    """Queries, latent cache and up-projections of a converted block (unit-variance logits)."""
    cfg = _cfg(case)
    rnd = _Draw(seed)
    B, T, H, dk, rkv = cfg.batch, cfg.seq, cfg.n_heads, cfg.head_dim, cfg.kv_rank
    n = B if case["kind"] == "decode" else B * T
    x = dict(cfg=cfg, q=rnd(n, H, cfg.qk_dim).to(BF), cache=rnd(B, T, rkv + cfg.rope_dim).to(BF),
             Wuk=rnd(cfg.s_kv_groups * cfg.nope_dim, rkv, std=rkv ** -0.5).to(BF),
             Wuv=rnd(cfg.s_kv_groups * dk, rkv, std=rkv ** -0.5).to(BF))
    if case["kind"] == "decode":
        lens = rnd.ints(max(1, T // 8), T, B) if case["ragged"] else torch.full((B,), T, device=DEV)
        x["lens"] = lens.to(torch.int32)
    else:
        x["Wo"] = rnd(cfg.hidden, H * dk, std=(H * dk) ** -0.5).to(BF)
    return x


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _ptr(t):
    return None if t is None else t.data_ptr()


def _buf(nbytes):
    assert nbytes > 0, L.last_error()
    return torch.empty(nbytes, dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("decode", "prefill"):
        s = _attend(case, seed)
        cfg = s["cfg"]
        s["c"] = c = L.make_cfg(cfg)
        if kind == "decode":
            s["o"] = torch.empty(cfg.batch, cfg.n_heads, cfg.head_dim, dtype=BF, device=DEV)
            if not case["noalloc"]:
                s["ws"] = _buf(L.mla_recon_decode_workspace_size(c, cfg.seq))
        else:
            s["ws"] = _buf(L.mla_recon_prefill_workspace_size(c))
            form = case["form"]
            s["o"] = (torch.empty(cfg.tokens, cfg.n_heads, cfg.head_dim, dtype=BF, device=DEV)
                      if "o" in form.split("+") else None)
            s["A"] = (torch.empty(cfg.tokens, cfg.hidden, dtype=torch.float32, device=DEV)
                      if form != "o" else None)
            s["fold"] = None
            if form == "folded":  # folded once, when the weights are loaded
                s["fold"] = torch.empty(cfg.hidden, cfg.n_heads * cfg.kv_rank, dtype=BF, device=DEV)
                L.mla_recon_fold_uv_into_o(c, _ptr(s["Wo"]), _ptr(s["Wuv"]), _ptr(s["fold"]), _stream())
        s["case"] = case
        return s
    s = _capture(case, seed) if kind == "capture" else _layer(case, seed)
    cfg = s["cfg"]
    s["case"], s["c"] = case, L.make_cfg(cfg)
    s["ws"] = _buf(L.mla_recon_workspace_size(s["c"]))
    tw = s["tw"]
    s["ctw"] = L.TeacherW(_ptr(tw["Wq"]), _ptr(tw["Wk"]), _ptr(tw["Wv"]), _ptr(tw["Wo"]), _ptr(s["inv_t"]))
    if kind in ("capture", "fourcall"):
        s["A_t"] = torch.empty(cfg.tokens, cfg.hidden, dtype=torch.float32, device=DEV)
    if kind == "capture":
        s["h_next"] = torch.empty_like(s["h"])
        return s
    sw = s["sw"]
    s["csw"] = L.StudentW(_ptr(sw["Wdq"]), _ptr(sw["Wuq"]), _ptr(sw["Wdkv_kr"]), _ptr(sw["Wuk"]),
                          _ptr(sw["Wuv"]), _ptr(s["inv_s"]))
    s["loss"] = torch.empty(2, dtype=torch.float32, device=DEV)
    s["grads"] = {n: torch.empty(sw["W" + n[2:]].shape, dtype=torch.float32, device=DEV)
                  for n in GRADS if sw["W" + n[2:]] is not None}
    s["cg"] = L.StudentGrads(*[_ptr(s["grads"].get(n)) for n in GRADS])
    if kind == "fourcall":
        s["A_s"] = torch.empty_like(s["A_t"])
        s["dA"] = torch.empty(cfg.tokens, cfg.hidden, dtype=BF, device=DEV)
    if kind == "train":
        s["step"] = OPT_STEP0
        s["master"] = {n: sw["W" + n[2:]].float() for n in s["grads"]}
        s["opt"] = [L.AdamwTensor(_ptr(s["master"][n]), _ptr(s["m"][n]), _ptr(s["v"][n]),
                                  _ptr(sw["W" + n[2:]]), _ptr(g), g.numel())
                    for n, g in s["grads"].items()]
        # the minibatch loop caches the frozen teacher's output once per minibatch
        L.mla_recon_teacher_cache(s["c"], _ptr(s["h"]), s["ctw"], _ptr(s["ws"]), s["ws"].numel(),
                                  _stream())
    return s


# ---- one pass ----------------------------------------------------------------------------
def run(s):
    case, c, st = s["case"], s["c"], _stream()
    kind = case["kind"]
    if kind == "decode":
        args = (c, _ptr(s["q"]), _ptr(s["cache"]), case["seq"], _ptr(s["lens"]), _ptr(s["Wuk"]),
                _ptr(s["Wuv"]), _ptr(s["o"]))
        if case["noalloc"]:
            L.mla_recon_decode_noalloc(*args, st)
        else:
            L.mla_recon_decode(*args, _ptr(s["ws"]), s["ws"].numel(), st)
        return dict(o=s["o"])
    if kind == "prefill":
        folded = s["fold"] is not None
        L.mla_recon_prefill(c, _ptr(s["q"]), _ptr(s["cache"]), _ptr(s["Wuk"]),
                            None if folded else _ptr(s["Wuv"]), None if folded else _ptr(s["Wo"]),
                            _ptr(s["fold"]), _ptr(s["o"]), _ptr(s["A"]), _ptr(s["ws"]),
                            s["ws"].numel(), st)
        return {k: s[k] for k in ("o", "A") if s[k] is not None}
    h, ws, wsb = _ptr(s["h"]), _ptr(s["ws"]), s["ws"].numel()
    if kind == "capture":
        cfg = s["cfg"]
        L.mla_recon_teacher_fwd(c, h, s["ctw"], _ptr(s["A_t"]), ws, wsb, st)
        L.mla_recon_residual_rmsnorm(_ptr(s["x"]), _ptr(s["A_t"]), _ptr(s["h_next"]), cfg.tokens,
                                     cfg.hidden, L.MLA_BF16, 1e-6, st)
        return dict(A_t=s["A_t"], x=s["x"], h=s["h_next"])
    Wo, mask, loss = _ptr(s["tw"]["Wo"]), _ptr(s["mask"]), _ptr(s["loss"])
    if kind == "step":
        L.mla_recon_step(c, h, s["ctw"], s["csw"], mask, loss, None, s["cg"], ws, wsb, st)
        return dict(loss=s["loss"], **s["grads"])
    if kind == "fourcall":
        A_t, A_s, dA = _ptr(s["A_t"]), _ptr(s["A_s"]), _ptr(s["dA"])
        L.mla_recon_teacher_fwd(c, h, s["ctw"], A_t, ws, wsb, st)
        L.mla_recon_student_fwd(c, h, s["csw"], Wo, A_s, ws, wsb, st)
        L.mla_recon_loss(c, A_s, A_t, mask, loss, dA, ws, wsb, st)
        L.mla_recon_bwd(c, h, s["csw"], Wo, dA, s["cg"], ws, wsb, st)
        return dict(loss=s["loss"], A_t=s["A_t"], A_s=s["A_s"], dA=s["dA"], **s["grads"])
    L.mla_recon_student_step(c, h, s["csw"], Wo, mask, loss, None, s["cg"], ws, wsb, st)
    s["step"] += 1
    L.mla_recon_adamw(s["opt"], L.MLA_BF16, s["step"], stream=st, **OPT)
    return dict(loss=s["loss"], grads=s["grads"], master=s["master"], m=s["m"], v=s["v"],
                w={n: s["sw"]["W" + n[2:]] for n in s["grads"]})


# ---- least work --------------------------------------------------------------------------
def work(case):
    cfg = _cfg(case)
    N, D, H, dk, rkv = cfg.tokens, cfg.hidden, cfg.n_heads, cfg.head_dim, cfg.kv_rank
    G, Gk, dn, dr, dqk = cfg.n_kv_groups, cfg.s_kv_groups, cfg.nope_dim, cfg.rope_dim, cfg.qk_dim
    kind = case["kind"]
    up = Gk * (dn + dk) * rkv
    if kind == "decode":
        # the filled cache rows (mean length of a ragged draw), every head against each row
        rows = case["batch"] * (case["seq"] * (0.5625 if case["ragged"] else 1.0))
        n = case["batch"]
        return dict(bytes=2.0 * (rows * (rkv + dr) + up + n * H * (dqk + dk)),
                    flops=2.0 * H * (rows * (2 * rkv + dr) + n * rkv * (dn + dk)))
    if kind == "prefill":
        f = cfg.flops()
        flops = f["S3_up_proj"] + f["S4_attn_fwd"]
        nbytes = 2.0 * (N * H * dqk + N * (rkv + dr) + up)
        if "o" in case["form"].split("+"):
            nbytes += 2.0 * N * H * dk
        if case["form"] != "o":
            nbytes += 4.0 * N * D + 2.0 * D * H * (rkv if case["form"] == "folded" else dk)
            flops += f["S5_wo"]
        return dict(bytes=nbytes, flops=flops)
    f = cfg.flops()
    t_w = 2.0 * D * dk * (2 * H + 2 * G)
    if kind == "capture":
        return dict(bytes=2.0 * N * D + t_w + N * D * (4.0 + 8.0 + 2.0),
                    flops=f["T1_qkv_proj"] + f["T3_attn_fwd"] + f["T4_wo"])
    n_s = ((cfg.q_rank or 0) * D + H * dqk * (cfg.q_rank or D) + cfg.kv_out * D + up)
    s_flops = sum(v for k, v in f.items() if k[0] in "SB" and k not in ("S5_wo", "B1_dO"))
    gram = 2.0 * (H * dk) ** 2 * (N + D)  # W_O^T W_O and its product with o_s - o_t
    wo = min(2.0 * f["T4_wo"], gram)      # or that difference through W_O and back
    if kind == "fourcall":
        return dict(bytes=2.0 * N * D + t_w + 6.0 * n_s + 10.0 * N * D, flops=cfg.total_flops())
    if kind == "train":
        return dict(bytes=2.0 * N * D + 2.0 * D * H * dk + n_s * (2.0 + 4.0 + 12.0 + 12.0 + 2.0),
                    flops=s_flops + wo)
    return dict(bytes=2.0 * N * D + t_w + 6.0 * n_s,
                flops=s_flops + f["T1_qkv_proj"] + f["T3_attn_fwd"] + wo)


# ---- tolerance ---------------------------------------------------------------------------
def tolerance(case):
    return TOL[case["kind"]]


# About four times the largest error of any output against `exact` over the listed and some
# drawn cases: gradients 1e-3 (long sequences) to 2.9e-3 (short ones), A and o 3e-3, dA (the
# rounded difference of two outputs) 4.1e-3, the loss 1e-4.
TOL = {
    "step": dict(rel=1.2e-2),
    "fourcall": dict(rel=1.6e-2),
    "train": dict(rel=1.2e-2),
    "capture": dict(rel=1.3e-2),
    "decode": dict(rel=1.2e-2),
    "prefill": dict(rel=1.2e-2),
}


# ---- float64 -----------------------------------------------------------------------------
def _d(x):
    return {k: None if v is None else v.double() for k, v in x.items()}


def _rope(x, inv, T, sign=1.0):
    """Rotate-half pairs (p, p + d/2) of x [B, T, heads, d] by t * inv[..., p]."""
    t = torch.arange(T, device=DEV, dtype=torch.float64)
    ang = t[:, None, None] * inv.double().reshape(-1, inv.shape[-1])[None]  # [T, 1 or heads, d/2]
    c, s = ang.cos(), sign * ang.sin()
    a, b = x.chunk(2, dim=-1)
    return torch.cat([a * c - b * s, a * s + b * c], dim=-1)


def _probs(q, k, scale):
    S = (q @ k.T) * scale
    T = S.shape[0]
    S.masked_fill_(torch.ones(T, T, dtype=torch.bool, device=DEV).triu_(1), -math.inf)
    return torch.softmax(S, dim=-1)


def _causal(q, k, v, scale):
    """o [B, T, H, dv]; k and v hold a head of the group count that divides H."""
    B, T, H, _ = q.shape
    o = torch.empty(B, T, H, v.shape[-1], dtype=torch.float64, device=DEV)
    for b in range(B):
        for i in range(H):
            P = _probs(q[b, :, i], k[b, :, i * k.shape[2] // H], scale)
            o[b, :, i] = P @ v[b, :, i * v.shape[2] // H]
    return o


def _teacher64(x):
    cfg, h, w = x["cfg"], x["h"].double(), _d(x["tw"])
    B, T, dk = cfg.batch, cfg.seq, cfg.head_dim
    inv = x["inv_t"][None]
    q = _rope((h @ w["Wq"].T).view(B, T, -1, dk), inv, T)
    k = _rope((h @ w["Wk"].T).view(B, T, -1, dk), inv, T)
    v = (h @ w["Wv"].T).view(B, T, -1, dk)
    return _causal(q, k, v, cfg.softmax_scale).reshape(cfg.tokens, -1)


def _step64(x):
    """o_t, A_s - A_t and everything after it: loss, gradients."""
    cfg, h, w = x["cfg"], x["h"].double(), _d(x["sw"])
    Wo = x["tw"]["Wo"].double()
    B, T, N, H, dk, rkv = cfg.batch, cfg.seq, cfg.tokens, cfg.n_heads, cfg.head_dim, cfg.kv_rank
    Gk, Gr, dn, dr, sc = (cfg.s_kv_groups, cfg.s_rope_groups, cfg.nope_dim, cfg.rope_dim,
                          cfg.softmax_scale)
    o_t = _teacher64(x)
    inv_h = x["inv_s"].repeat_interleave(H // Gr, 0)
    cq = h if w["Wdq"] is None else h @ w["Wdq"].T
    q = (cq @ w["Wuq"].T).view(B, T, H, dn + dr)
    q = torch.cat([q[..., :dn], _rope(q[..., dn:], inv_h, T)], -1)
    ckv = h @ w["Wdkv_kr"].T
    c = ckv[:, :rkv]
    kpe = _rope(ckv[:, rkv:].view(B, T, Gr, dr), x["inv_s"], T)
    kn = (c @ w["Wuk"].T).view(B, T, Gk, dn)
    v = (c @ w["Wuv"].T).view(B, T, Gk, dk)
    k = torch.cat([kn, kpe.repeat_interleave(Gk // Gr, 2)], -1)
    o = _causal(q, k, v, sc).reshape(N, -1)
    M = x["mask"].double()[:, None]
    A_t, A_s = o_t @ Wo.T, o @ Wo.T
    E = M * (A_s - A_t)
    den = cfg.hidden * M.sum()
    loss = torch.stack([E.square().sum() / den, E.square().sum() / (M * A_t).square().sum()])
    dA = 2.0 * E / den
    dO = (dA @ Wo).view(B, T, H, dk)
    dq, dk_, dv = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for b in range(B):
        for i in range(H):
            g = i * Gk // H
            P = _probs(q[b, :, i], k[b, :, g], sc)
            dv[b, :, g] += P.T @ dO[b, :, i]
            dP = dO[b, :, i] @ v[b, :, g].T
            dS = P * (dP - (dP * P).sum(-1, keepdim=True)) * sc
            dq[b, :, i] = dS @ k[b, :, g]
            dk_[b, :, g] += dS.T @ q[b, :, i]
    dq = torch.cat([dq[..., :dn], _rope(dq[..., dn:], inv_h, T, -1.0)], -1).reshape(N, -1)
    dkpe = dk_[..., dn:].reshape(B, T, Gr, Gk // Gr, dr).sum(3)
    dkpe = _rope(dkpe, x["inv_s"], T, -1.0).reshape(N, -1)
    dkn, dv = dk_[..., :dn].reshape(N, -1), dv.reshape(N, -1)
    dc = dkn @ w["Wuk"] + dv @ w["Wuv"]
    grads = dict(dWuq=dq.T @ cq, dWdkv_kr=torch.cat([dc, dkpe], -1).T @ h, dWuk=dkn.T @ c,
                 dWuv=dv.T @ c)
    if w["Wdq"] is not None:
        grads["dWdq"] = (dq @ w["Wuq"]).T @ h
    return dict(loss=loss, A_t=A_t, A_s=A_s, dA=dA, grads=grads)


def _attend64(x, rows_of):
    """o [rows, H, d_k]; rows_of(b): the query rows of sequence b and, for each, its last key."""
    cfg = x["cfg"]
    H, Gk, dn, rkv, dk = cfg.n_heads, cfg.s_kv_groups, cfg.nope_dim, cfg.kv_rank, cfg.head_dim
    q, cache, Wuk, Wuv = (x[n].double() for n in ("q", "cache", "Wuk", "Wuv"))
    o = torch.zeros(q.shape[0], H, dk, dtype=torch.float64, device=DEV)
    for b in range(cfg.batch):
        c, kpe = cache[b, :, :rkv], cache[b, :, rkv:]
        kn = (c @ Wuk.T).view(-1, Gk, dn)
        v = (c @ Wuv.T).view(-1, Gk, dk)
        rows, last = rows_of(b)
        past = torch.arange(cfg.seq, device=DEV)[None, :] > last[:, None]
        for i in range(H):
            g = i * Gk // H
            k = torch.cat([kn[:, g], kpe], -1)
            S = (q[rows, i] @ k.T) * cfg.softmax_scale
            o[rows, i] = torch.softmax(S.masked_fill_(past, -math.inf), -1) @ v[:, g]
    return o


def exact(case, seed):
    kind = case["kind"]
    if kind == "decode":
        x = _attend(case, seed)
        return dict(o=_attend64(x, lambda b: (torch.tensor([b], device=DEV),
                                              x["lens"][b:b + 1].long() - 1)))
    if kind == "prefill":
        x = _attend(case, seed)
        T = case["seq"]
        t = torch.arange(T, device=DEV)
        o = _attend64(x, lambda b: (b * T + t, t))
        out = {}
        if "o" in case["form"].split("+"):
            out["o"] = o
        if case["form"] != "o":
            out["A"] = o.reshape(o.shape[0], -1) @ x["Wo"].double().T
        return out
    if kind == "capture":
        x = _capture(case, seed)
        A = _teacher64(x) @ x["tw"]["Wo"].double().T
        y = x["x"].double() + A
        return dict(A_t=A, x=y, h=y * torch.rsqrt(y.square().mean(-1, keepdim=True) + 1e-6))
    x = _layer(case, seed)
    r = _step64(x)
    if kind == "fourcall":
        return dict(loss=r["loss"], A_t=r["A_t"], A_s=r["A_s"], dA=r["dA"], **r["grads"])
    r["loss"][1] = math.nan  # the single call leaves the relative error out
    if kind == "step":
        return dict(loss=r["loss"], **r["grads"])
    out = dict(loss=r["loss"], grads=r["grads"], master={}, m={}, v={}, w={})
    b1, b2, n = OPT["beta1"], OPT["beta2"], OPT_STEP0 + 1
    for name, g in r["grads"].items():
        w = x["sw"]["W" + name[2:]].double()
        m = b1 * x["m"][name].double() + (1 - b1) * g
        v = b2 * x["v"][name].double() + (1 - b2) * g * g
        upd = (m / (1 - b1 ** n)) / ((v / (1 - b2 ** n)).sqrt() + OPT["eps"])
        w = w - OPT["lr"] * (upd + OPT["weight_decay"] * w)
        out["master"][name], out["m"][name], out["v"][name], out["w"][name] = w, m, v, w
    return out
