"""The work that a program built on this package has it do, as cases that can be timed and compared.

A case names one public entry point and its sizes.  The model shapes are the package's own: the
7B-shaped backbone (hidden 4096, 32 heads of 128, MLP 11008) of all workloads but the smallest, and
the small one (hidden 256, 4 heads of 64, MLP 1024); a middle one (hidden 1024) stands for what
lies between.  Token counts are those of the workloads (256 image and 256 point tokens a view,
16 to 64 language tokens) and, in drawn cases, anything between a few tokens and the largest batch.

Kinds:
  call         PrefillPlan.run: a whole pruned prefill
  layer        Context.prefill_layer: one backbone layer on kept tokens, gathered position ids
  score_layer  Context.prefill_layer_salience: the last full-sequence layer, which scores the tokens
  score_pass   Context.score_only: the scoring alone, for pruning before any layer
  prune        Context.prune_step: salience, budget, selection and gather from given attention rows
  select       Context.modality_budget + select_topk: what a smoothed episode calls on its state
  indicators   Context.salience + feature_share + modality_decompose: the per-patch indicators
  masks        Context.candidate_masks + mask_indices: the retention masks of an episode step
"""
import math

import torch

from paper_2604_09244_amd import binding as mv
from paper_2604_09244_amd import workloads as W

MODELS = {  # hidden size, heads, head dim, MLP width
    "7b": (4096, 32, 128, 11008),
    "mid": (1024, 8, 128, 2816),
    "small": (256, 4, 64, 1024),
}
DEV = "cuda"


# ---- the cases ------------------------------------------------------------------------------
def listed():
    return [
        # the smallest whole prefill: one small layer, pruning before it; launches and latency
        dict(name="call_tiny", kind="call", model="small", B=1, n2=64, n3=64, nt=16, L=1, p=0),
        # one robot, one view, 512 visual tokens: the interactive call, four 7B-shaped layers
        dict(name="call_single_view", kind="call", model="7b", B=1, n2=256, n3=256, nt=32, L=4, p=2),
        # a layer on the kept tokens of that call (40 % of 512, and 32 language tokens)
        dict(name="layer_1x237", kind="layer", model="7b", B=1, S=237),
        # the same for four episodes side by side
        dict(name="layer_4x237", kind="layer", model="7b", B=4, S=237),
        # eight samples of a three-camera, four-sweep scene at 30 %: rows that fill no tile evenly
        dict(name="layer_8x586", kind="layer", model="7b", B=8, S=586),
        # the benchmark's batch at 50 %: 30 of its 32 layers run at this size
        dict(name="layer_16x1344", kind="layer", model="7b", B=16, S=1344),
        # the benchmark's scoring layer on all tokens: the largest single call
        dict(name="score_layer_16x2624", kind="score_layer", model="7b", B=16, n2=512, n3=2048, nt=64),
        # the scoring pass when masks go back to the encoder (pruning before any layer)
        dict(name="score_pass_1x544", kind="score_pass", model="7b", B=1, S=544, nt=32),
        # the pruning step of the benchmark's batch from written attention rows, keep 50 %
        dict(name="prune_16x2624", kind="prune", model="7b", B=16, n2=512, n3=2048, nt=64, keep=500),
        # budget and per-modality top-k on smoothed scores, eight samples, keep 30 %
        dict(name="select_8x1792", kind="select", model="7b", B=8, n2=768, n3=1024, nt=48, keep=300),
        # the indicators of an action-iteration step, four episodes
        dict(name="indicators_4x256", kind="indicators", model="7b", B=4, P=256, nt=32),
        # the masks of that step
        dict(name="masks_4x256", kind="masks", model="7b", B=4, P=256, nt=32),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    kind = rng.choice(["call", "layer", "layer", "layer", "score_layer", "score_pass", "prune", "select",
                       "indicators", "masks"])
    model = rng.choice(["7b", "7b", "7b", "mid", "small"])
    nt = rng.randint(8, 64)
    B = _log_int(rng, 1, 16)
    if kind == "call":
        c = dict(model=model, B=min(B, 4), n2=_log_int(rng, 16, 512), n3=_log_int(rng, 16, 512), nt=nt,
                 L=rng.randint(1, 3))
        c["p"] = rng.randint(0, min(2, c["L"]))
    elif kind == "layer":
        c = dict(model=model, B=B, S=_log_int(rng, 24, 2048))
    elif kind == "score_layer":
        c = dict(model=model, B=B, n2=_log_int(rng, 16, 768), n3=_log_int(rng, 16, 1800), nt=nt)
    elif kind == "score_pass":
        c = dict(model=model, B=min(B, 8), S=nt + _log_int(rng, 32, 2500), nt=nt)
    elif kind == "prune":
        c = dict(model=model, B=B, n2=_log_int(rng, 16, 768), n3=_log_int(rng, 16, 1700), nt=nt,
                 keep=rng.randint(150, 1000))
    elif kind == "select":
        c = dict(model=model, B=B, n2=_log_int(rng, 16, 16384), n3=_log_int(rng, 16, 16384), nt=nt,
                 keep=rng.randint(150, 1000))
    elif kind == "indicators":
        c = dict(model=model, B=min(B, 8), P=_log_int(rng, 16, 1024), nt=nt)
    else:
        c = dict(model=model, B=B, P=_log_int(rng, 16, 4096), nt=nt)
    c["kind"] = kind
    return c


# ---- inputs -----------------------------------------------------------------------------------
def _workload(case, seed):
    """The package's description of the inputs: token counts, distributions, and the seed."""
    D, H, dh, F = MODELS[case["model"]]
    kind = case["kind"]
    if kind == "layer":
        n2, n3, nt = case["S"] // 2, case["S"] - case["S"] // 2, 0
    elif kind == "score_pass":
        n2 = (case["S"] - case["nt"]) // 2
        n3, nt = case["S"] - case["nt"] - n2, case["nt"]
    elif kind in ("indicators", "masks"):
        n2, n3, nt = case["P"], case["P"], case["nt"]
    else:
        n2, n3, nt = case["n2"], case["n3"], case["nt"]
    keep = case.get("keep", 500)
    return W.Workload(kind, L=case.get("L", 1), D=D, H=H, dh=dh, F=F, n2=n2, n3=n3, nt=nt,
                      keep_permille=keep, B=case["B"], p=case.get("p", 0), seed=seed % 1000003,
                      offsets=case["model"] != "small", heavy_tail=True)


def _hidden(wl):
    """Hidden states and position ids; rows of a layer on kept tokens carry ids with gaps."""
    x, pos = W.hidden_states(wl, device=DEV)
    if wl.name == "layer":
        g = torch.Generator().manual_seed(wl.seed + 77)
        rows = [torch.randperm(2 * wl.S, generator=g)[:wl.S].sort().values for _ in range(wl.B)]
        pos = torch.stack(rows).to(torch.int32).to(DEV)
    return x, pos


def _bias(wl):
    """Scoring bias.  In a whole call the image tokens as a group carry the attention and the budget
    is their number, so that which tokens are kept does not hang on a rounding: every later value
    of the call depends on that set."""
    kb = W.scoring_bias(wl, device=DEV)
    if wl.name == "call":
        kb[:, :wl.n2] += 12.0
    return kb


def _weights(wl):
    return [W.layer_weights(wl, l, device=DEV) for l in range(wl.L)]


def _rope_len(wl):
    return 2 * wl.S if wl.name == "layer" else wl.S


def _features(wl):
    """Token features whose 3D part is the weaker one, as in the paper's measurements."""
    x, _ = W.hidden_states(wl, device=DEV)
    return W.weaken_3d(wl, x)


def prepare(case, seed):
    wl = _workload(case, seed)
    kind = case["kind"]
    s = dict(kind=kind, wl=wl)
    # (a workspace for layers only where a layer runs)
    D, F = (wl.D, wl.F) if kind in ("call", "layer", "score_layer", "score_pass") else (64, 64)
    ctx = mv.Context(wl.B, wl.S, D, wl.H, F, max(wl.nt, 1))
    cfg = mv.LayerCfg(wl.D, wl.H, wl.dh, wl.F, wl.rms_eps)
    s.update(ctx=ctx, cfg=cfg)
    bf, i32, f32 = torch.bfloat16, torch.int32, torch.float32
    if kind in ("call", "layer", "score_layer", "score_pass"):
        s["x"], s["pos"] = _hidden(wl)
        packed = [mv.pack_layer(w) for w in _weights(wl)]
        if kind == "call":
            s["plan"] = mv.PrefillPlan(ctx, cfg, packed, wl.B, wl.n2, wl.n3, wl.nt, wl.n2, wl.p)
        else:
            rope = ctx.rope_table(wl.rope_base, _rope_len(wl), wl.dh)
            s["layer"] = ctx.layer_struct(packed[0], rope)
            s["y"] = torch.empty_like(s["x"])
        if kind != "layer":
            s["bias"] = _bias(wl)
        if kind == "score_layer":
            s["sal"] = torch.empty(wl.B, wl.n_vis, dtype=f32, device=DEV)
        if kind == "score_pass":
            s["probs"] = torch.empty(wl.B, wl.H, wl.nt, wl.S, dtype=f32, device=DEV)
    elif kind == "prune":
        s["x"], s["pos"] = W.hidden_states(wl, device=DEV)
        s["attn"] = W.synthetic_probs(wl, device=DEV)
        s["out"] = dict(sal=torch.empty(wl.B, wl.n_vis, dtype=f32, device=DEV),
                        k2k3=torch.empty(wl.B, 2, dtype=i32, device=DEV),
                        kept_idx=torch.empty(wl.B, wl.S_kept, dtype=i32, device=DEV),
                        h=torch.empty(wl.B, wl.S_kept, wl.D, dtype=bf, device=DEV),
                        pos=torch.empty(wl.B, wl.S_kept, dtype=i32, device=DEV))
    elif kind == "select":
        s["score"] = W.synthetic_salience(wl, device=DEV)
        s["k2k3"] = torch.empty(wl.B, 2, dtype=i32, device=DEV)
        s["kept"] = torch.empty(wl.B, wl.S_kept, dtype=i32, device=DEV)
    elif kind == "indicators":
        s["attn"] = W.synthetic_probs(wl, device=DEV)
        s["feat"] = _features(wl)
        s["sal"] = torch.empty(wl.B, wl.n_vis, dtype=f32, device=DEV)
        s["ind"] = torch.empty(4, wl.B, wl.n2, dtype=f32, device=DEV)
    else:
        s["x_hat"] = W.synthetic_indicators(wl, device=DEV, seed=wl.seed)
        s["sal"] = W.synthetic_salience(wl, device=DEV)
        s["u"] = W.uniform_draws(wl, device=DEV)
        s["masks"] = tuple(torch.empty(wl.B, wl.n2, dtype=torch.uint8, device=DEV) for _ in range(3))
        s["len"] = torch.empty(wl.B, dtype=i32, device=DEV)
        s["kept"] = torch.empty(wl.B, wl.S, dtype=i32, device=DEV)
    return s


# ---- one pass -----------------------------------------------------------------------------------
def run(state):
    s, kind, wl, ctx = state, state["kind"], state["wl"], state["ctx"]
    if kind == "call":
        plan = s["plan"]
        y = plan.run(s["x"], s["pos"], s["bias"], on_the_fly=wl.p >= 1)
        return dict(y=y, sal=plan.prune["sal"], kept=plan.prune["kept_idx"], pos=plan.prune["pos"])
    if kind == "layer":
        return dict(y=ctx.prefill_layer(s["cfg"], s["layer"], s["x"], s["pos"], s["y"]))
    if kind == "score_layer":
        y, sal = ctx.prefill_layer_salience(s["cfg"], s["layer"], s["x"], s["pos"], wl.nt, wl.n_vis,
                                            y=s["y"], key_bias=s["bias"], sal=s["sal"])
        return dict(y=y, sal=sal)
    if kind == "score_pass":
        return dict(probs=ctx.score_only(s["cfg"], s["layer"], s["x"], s["pos"], wl.nt, s["bias"],
                                         s["probs"]))
    if kind == "prune":
        return dict(ctx.prune_step(s["attn"], s["x"], s["pos"], wl.n2, wl.n3, wl.nt, wl.k_total,
                                   out=s["out"]))
    if kind == "select":
        k2k3 = ctx.modality_budget(s["score"], wl.n2, wl.n3, wl.k_total, out=s["k2k3"])
        kept = ctx.select_topk(s["score"], k2k3, wl.n2, wl.n3, wl.nt, wl.k_total, out=s["kept"])
        return dict(k2k3=k2k3, kept=kept)
    if kind == "indicators":
        sal = ctx.salience(s["attn"], wl.n_vis, out=s["sal"])
        ctx.feature_share(s["feat"], wl.n2, out=(s["ind"][0], s["ind"][1]))
        ctx.modality_decompose(s["attn"], wl.n2, out=(s["ind"][2], s["ind"][3]))
        return dict(sal=sal, ind=s["ind"])
    m2, m3, sem, length = ctx.candidate_masks(s["x_hat"], s["sal"], s["u"], wl.nt,
                                              out=(*s["masks"], s["len"]))
    kept = ctx.mask_indices(m2, m3, wl.nt, wl.S, out=s["kept"])
    return dict(mask2d=m2, mask3d=m3, sem=sem, length=length, kept=kept)


# ---- what a pass cannot do without -----------------------------------------------------------------
def _layer_work(wl, rows):
    """One layer on B samples of `rows` tokens: weights once, activations in and out."""
    D, F, M = wl.D, wl.F, wl.B * rows
    weights = 4 * D * D + 3 * D * F
    flops = 2.0 * M * weights + 2.0 * wl.B * D * rows * (rows + 1)
    return 2.0 * weights + 4.0 * M * D, flops


def work(case):
    wl = _workload(case, 0)
    kind, B, D = case["kind"], wl.B, wl.D
    score_flops = 2.0 * B * wl.nt * wl.S * D
    if kind == "layer":
        b, f = _layer_work(wl, wl.S)
    elif kind == "score_layer":
        b, f = _layer_work(wl, wl.S)
        b, f = b + 4.0 * B * wl.n_vis, f + score_flops
    elif kind == "call":
        bf_, ff = _layer_work(wl, wl.S)
        bk, fk = _layer_work(wl, wl.n2 + wl.nt)
        b, f = wl.p * bf_ + (wl.L - wl.p) * bk, wl.p * ff + (wl.L - wl.p) * fk + score_flops
        if wl.p == 0:   # keys of every row, queries of the scoring rows
            b, f = b + 4.0 * D * D + 2.0 * B * wl.S * D, f + 2.0 * B * (wl.S + wl.nt) * D * D
    elif kind == "score_pass":
        b = 4.0 * D * D + 2.0 * B * wl.S * D + 4.0 * B * wl.H * wl.nt * wl.S
        f = 2.0 * B * (wl.S + wl.nt) * D * D + score_flops
    elif kind == "prune":
        b = 4.0 * B * wl.H * wl.nt * wl.n_vis + 4.0 * B * wl.n_vis + 4.0 * B * wl.S_kept * (D + 3)
        f = 1.0 * B * wl.H * wl.nt * wl.n_vis
    elif kind == "select":
        b, f = 4.0 * B * (wl.n_vis + wl.S_kept), 1.0 * B * wl.n_vis
    elif kind == "indicators":
        b = 4.0 * B * wl.H * wl.nt * wl.n_vis + 2.0 * B * wl.n_vis * D + 4.0 * B * 6 * wl.n2
        f = 8.0 * B * wl.H * wl.nt * wl.n_vis + 1.0 * B * wl.n_vis * D
    else:
        b, f = 4.0 * B * wl.n2 * 6 + 3.0 * B * wl.n2 + 4.0 * B * wl.S, 20.0 * B * wl.n2
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times what a pass differs from exact(): bf16 operands and a bf16 output put a layer
    0.0036 (relative, 2-norm) and its worst element 0.025 root mean squares off, four layers one
    after the other 0.0073; scoring probabilities from bf16 queries and keys are 0.0012 off as a
    whole and about 1 % each.  The pruning step and the indicators are 32-bit sums (1e-7 measured);
    selection and masks are whole numbers."""
    kind = case["kind"]
    if kind in ("select", "masks"):
        return "exact"
    if kind in ("prune", "indicators"):
        return {"rel": 1e-5, "max": 1e-4}
    if kind == "score_pass":
        return {"rel": 0.005, "max": 0.2}
    if kind == "call":
        return {"rel": 0.03, "max": 0.3}
    return {"rel": 0.015, "max": 0.15}


# ---- the same in 64 bits ------------------------------------------------------------------------
def _norm64(x, gain, eps):
    return x * gain.double() / torch.sqrt((x * x).mean(-1, keepdim=True) + eps)


def _rotate64(t, pos, base):
    """t [rows, H, dh], pos [rows]: pairs (i, i + dh/2) turned by pos * base^(-2i/dh)."""
    dh = t.shape[-1]
    inv = base ** (-torch.arange(dh // 2, dtype=torch.float64, device=t.device) / (dh // 2))
    ang = pos.double()[:, None] * inv
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = t[..., :dh // 2], t[..., dh // 2:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _probs64(q, k, row0, bias=None):
    """softmax(q k^T / sqrt(dh) + bias) of query rows row0.. over the keys up to each row: [H, nq, S]."""
    nq, S = q.shape[0], k.shape[0]
    lg = torch.matmul(q.transpose(0, 1), k.permute(1, 2, 0).contiguous()) / math.sqrt(q.shape[-1])
    if bias is not None:
        lg = lg + bias.double()[None, None]
    rows = row0 + torch.arange(nq, device=q.device)
    lg.masked_fill_(torch.arange(S, device=q.device)[None, :] > rows[:, None], -math.inf)
    return torch.softmax(lg, -1)


def _layer64(wl, w, x, pos, nt=0, bias=None):
    """One sample through one layer: (output rows, scoring probabilities of the last nt rows)."""
    w = {k: v.double() for k, v in w.items()}
    S, H, dh = x.shape[0], wl.H, wl.dh
    u = _norm64(x, w["g_attn"], wl.rms_eps)
    q = _rotate64((u @ w["wq"].T).view(S, H, dh), pos, wl.rope_base)
    k = _rotate64((u @ w["wk"].T).view(S, H, dh), pos, wl.rope_base)
    v = (u @ w["wv"].T).view(S, H, dh)
    scored = _probs64(q[S - nt:], k, S - nt, bias) if nt else None
    out = torch.empty_like(q)
    for r in range(0, S, 512):
        e = min(S, r + 512)
        p = _probs64(q[r:e], k[:e], r)
        out[r:e] = torch.matmul(p, v[:e].transpose(0, 1).contiguous()).transpose(0, 1)
    x1 = x + out.reshape(S, -1) @ w["wo"].T
    t = _norm64(x1, w["g_mlp"], wl.rms_eps)
    g = t @ w["w_gate"].T
    act = g * torch.sigmoid(g) * (t @ w["w_up"].T)
    return x1 + act @ w["w_down"].T, scored


def _score64(wl, w, x, pos, nt, bias):
    S, H, dh = x.shape[0], wl.H, wl.dh
    u = _norm64(x, w["g_attn"], wl.rms_eps)
    q = _rotate64((u[S - nt:] @ w["wq"].double().T).view(nt, H, dh), pos[S - nt:], wl.rope_base)
    k = _rotate64((u @ w["wk"].double().T).view(S, H, dh), pos, wl.rope_base)
    return _probs64(q, k, S - nt, bias)


def _select64(sal, wl, k_total):
    """Budget by mass and top-k per segment; of equal scores the lower index is kept."""
    m2 = float(sal[:wl.n2].sum() / sal.sum())
    k2 = min(max(int(math.floor(k_total * m2 + 0.5)), max(0, k_total - wl.n3)), min(wl.n2, k_total))
    a = torch.sort(sal[:wl.n2], descending=True, stable=True).indices[:k2].sort().values
    b = torch.sort(sal[wl.n2:], descending=True, stable=True).indices[:k_total - k2].sort().values
    text = torch.arange(wl.n_vis, wl.S, device=sal.device)
    return torch.cat([a, wl.n2 + b, text])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("select", "masks"):
        return None
    wl = _workload(case, seed)
    if kind in ("prune", "indicators"):
        p = W.synthetic_probs(wl, device=DEV)
        sal = torch.stack([r.double().sum((0, 1)) for r in p])[:, :wl.n_vis] / (wl.H * wl.nt)
        if kind == "prune":
            x, pos = W.hidden_states(wl, device=DEV)
            kept = torch.stack([_select64(r, wl, wl.k_total) for r in sal])
            h = torch.stack([x[b, kept[b]] for b in range(wl.B)])
            return dict(sal=sal, k2k3=None, kept_idx=kept, h=h.double(), pos=pos.gather(1, kept))
        P = wl.n2
        f = _features(wl).double().abs().sum(-1)
        l2, l3 = f[:, :P], f[:, P:2 * P]
        a = p.double().reshape(wl.B, -1, wl.S)
        a2, a3 = a[:, :, :P], a[:, :, P:2 * P]
        c = (a2 * a3).sum(1) / (a2 * a2).sum(1)
        n2, n3 = a2.abs().sum(1), a3.abs().sum(1)
        rest = (a3 - c[:, None] * a2).abs().sum(1)
        return dict(sal=sal, ind=torch.stack([l2 / (l2 + l3), l3 / (l2 + l3), n2 / (n2 + n3),
                                              rest / (n2 + n3)]))
    x, pos = _hidden(wl)
    ws = _weights(wl)
    if kind == "layer":
        return dict(y=torch.stack([_layer64(wl, ws[0], x[b].double(), pos[b])[0] for b in range(wl.B)]))
    bias = _bias(wl)
    if kind == "score_pass":
        return dict(probs=torch.stack([_score64(wl, ws[0], x[b].double(), pos[b], wl.nt, bias[b])
                                       for b in range(wl.B)]))
    ys, sals, keeps, ps = [], [], [], []
    for b in range(wl.B):
        h, ps_b = x[b].double(), pos[b]
        if kind == "score_layer":
            h, pr = _layer64(wl, ws[0], h, ps_b, wl.nt, bias[b])
        else:
            if wl.p == 0:
                pr = _score64(wl, ws[0], h, ps_b, wl.nt, bias[b])
            for l in range(wl.p):
                last = l == wl.p - 1
                h, got = _layer64(wl, ws[l], h, ps_b, wl.nt if last else 0, bias[b] if last else None)
                pr = got if last else None
        sal = pr.sum((0, 1))[:wl.n_vis] / (wl.H * wl.nt)
        if kind == "call":
            kept = _select64(sal, wl, wl.n2)
            h, ps_b = h[kept], ps_b[kept]
            for l in range(wl.p, wl.L):
                h, _ = _layer64(wl, ws[l], h, ps_b)
            keeps.append(kept)
            ps.append(ps_b)
        ys.append(h)
        sals.append(sal)
    out = dict(y=torch.stack(ys), sal=torch.stack(sals))
    if kind == "call":
        out.update(kept=torch.stack(keeps), pos=torch.stack(ps))
    return out
