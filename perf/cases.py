"""Workloads that time the checkpoint library through its public calls.

A case is one call of the Store / Load path as a serving engine makes it: pack after a
prefill, restore on a prefix hit, and Load with refresh (restore plus a replay of the
last W tokens) for the requests that refresh.  Shapes are those of `workloads/synth.py`
and of the tests: Kimi-Linear-shaped KDA layers (32 heads of 128 x 128, 38% of the rows
kept), the 24-layer model set with T = 8 rank slices, Qwen3-Next-shaped GDN layers
(16 key heads, 32 value heads, 12 kept per layer), the windows W of 16 to 2048 tokens,
and the smaller head sizes the refresh also takes.  Decay rates stand for model weights,
so the plan of a case is fixed; states, slots and suffix inputs come from the seed.
"""

import functools
import math

import numpy as np
import torch

import paper_2608_30386_amd as D


def listed():
    kda = dict(arch="kda", L=1, H=32, Hqk=32, dk=128, dv=128, T=1)
    model = dict(arch="kda", L=24, H=32, Hqk=32, dk=128, dv=128)
    gdn = dict(arch="gdn", L=3, H=32, Hqk=16, dk=128, dv=128, T=1)
    return [
        # one request's state of one layer is stored: the smallest call, all latency
        dict(name="store_one", kind="pack", n=1, keep="topk", **kda),
        # a batch of whole-model checkpoints stored into T = 8 rank slices: the largest Store
        dict(name="store_model", kind="pack", n=64, keep="wmax", w_max=1024, T=8, **model),
        # the same checkpoints loaded back without refresh: the largest Load
        dict(name="load_model", kind="restore", n=64, keep="wmax", w_max=1024, T=8, **model),
        # INT8 checkpoints of a few requests, an odd count, W_max = 64 keeps most rows
        dict(name="store_q8", kind="pack_q8", n=11, keep="wmax", w_max=64, T=1, **model),
        dict(name="load_q8", kind="restore_q8", n=11, keep="wmax", w_max=64, T=1, **model),
        # a prefix hit of a single request: fused Load with refresh at W_max = 128
        dict(name="hit_kda_one", kind="load_refresh", n=1, W=128, keep="topk", init="restored", **kda),
        # the headline Load with refresh: 16 requests x 32 heads, W = 1024
        dict(name="hit_kda_batch", kind="load_refresh", n=16, W=1024, keep="topk", init="restored", **kda),
        # refresh of states already restored: ragged window, odd batch, long horizon of history
        dict(name="refresh_kda_ragged", kind="refresh", n=5, W=777, keep="topk", init="zero", **kda),
        # the longest window of the serving shape
        dict(name="refresh_kda_long", kind="refresh", n=16, W=2048, keep="topk", init="restored", **kda),
        # one GDN layer of the headline GDN batch, fused Load with refresh
        dict(name="hit_gdn_batch", kind="load_refresh", n=8, W=1024, keep="topk", init="restored", **gdn),
        # GDN refresh of a small ragged batch
        dict(name="refresh_gdn_ragged", kind="refresh", n=3, W=517, keep="topk", init="zero", **gdn),
        # heads of another size (the per-column fp32 kernel): 64 x 64
        dict(name="refresh_d64", kind="refresh", n=8, W=512, keep="topk", init="restored",
             arch="kda", L=1, H=16, Hqk=16, dk=64, dv=64, T=1),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: kinds, architectures, head counts (32 heads, or one tensor-parallel
    rank's share of them), batch sizes and windows, log-uniform, odd values included."""
    kind = rng.choice(["pack", "restore", "pack_q8", "restore_q8"] + ["refresh", "load_refresh"] * 4)
    arch = rng.choice(["kda", "kda", "gdn"])
    H = rng.choice([4, 8, 16, 32, 32])
    c = dict(kind=kind, arch=arch, H=H, Hqk=H if arch == "kda" else H // 2, dk=128, dv=128, T=1)
    if "refresh" not in kind:
        c["L"] = _logint(rng, 1, 24)
        c["n"] = _logint(rng, 1, max(1, min(64, 64 * 24 * 32 // (c["L"] * H))))
        if kind in ("pack", "restore"):
            c["T"] = rng.choice([1, 2, 8])
        c.update(rng.choice([dict(keep="topk"), dict(keep="wmax", w_max=rng.choice([16, 64, 128, 512, 1024]))]))
        return c
    c["L"] = rng.choice([1, 2, 3])
    c["n"] = rng.randint(1, 16)
    c["W"] = _logint(rng, 16, 2048)
    c["init"] = rng.choice(["restored", "zero"])
    c["keep"] = "topk"
    if kind == "refresh" and rng.random() < 0.25:      # other head sizes
        c["dk"] = rng.choice([16, 32, 64])
        c["dv"] = rng.choice([16, 32, 64, 64, 100, 128])
        c["H"] = min(H, 16)
        c["Hqk"] = c["H"] if arch == "kda" else c["H"] // 2
        c["W"] = _logint(rng, 16, 512)
    return c


# ---- plan (fixed per model) -----------------------------------------------------------

@functools.lru_cache(maxsize=4)
def _plan(arch, L, H, Hqk, dk, dv, keep, w_max, T):
    sh = D.Shape(arch, L, H, Hqk, dk, dv)
    lam = np.random.default_rng([L, H, dk, arch == "gdn"]).uniform(
        math.log(1e-4), 0.0, size=(L, H, dk) if arch == "kda" else (L, H))
    g = D.dasc_static_log_decay(lam)
    if keep == "wmax":
        p = D.dasc_plan(sh, g, "threshold", 0, w_max, T)
    else:
        units = H * dk if arch == "kda" else H
        p = D.dasc_plan(sh, g, "topk_layer", round((0.38 if arch == "kda" else 0.375) * units), 1024, T)
    return sh, p, np.exp(lam)


def _plan_of(c):
    return _plan(c["arch"], c["L"], c["H"], c["Hqk"], c["dk"], c["dv"], c["keep"], c.get("w_max", 0), c["T"])


# ---- inputs -----------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _layer(c):
    return c["L"] - 1


def prepare(case, seed):
    sh, p, lam = _plan_of(case)
    gen, n, R, dv, T = _gen(seed), case["n"], int(p["n_rows"]), sh.dv, case["T"]
    C = int(p["slice_rows"])
    n_slots = n + 3                                     # pools hold more slots than the batch
    kind = case["kind"]

    def i32(a):
        return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.int32, device="cuda")

    def slots():
        return torch.randperm(n_slots, generator=gen, device="cuda")[:n].to(torch.int32)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda").mul_(0.05)

    s = dict(kind=kind, sh=sh, n_rows=R, T=T, C=C, src=slots(), dst=slots(),
             unit_row=i32(p["unit_row"]), inv_row=i32(p["inv_row"]))
    pool = (n_slots, sh.n_layers, sh.n_heads, sh.dk, dv)
    if kind == "pack":
        s["states"] = normal(*pool)
        s["ckpt"] = torch.zeros((T, n_slots, C, dv), device="cuda")
    elif kind == "restore":
        s["ckpt"] = normal(T, n_slots, C, dv)
        s["states"] = torch.zeros(pool, device="cuda")
    elif kind == "pack_q8":
        s["states"] = normal(*pool)
        s["q"] = torch.zeros((n_slots, R, dv), dtype=torch.int8, device="cuda")
        s["scale"] = torch.zeros((n_slots, R), device="cuda")
    elif kind == "restore_q8":
        s["q"] = torch.randint(-127, 128, (n_slots, R, dv), generator=gen, device="cuda", dtype=torch.int8)
        s["scale"] = normal(n_slots, R).abs_().mul_(4.0 / 127.0)
        s["states"] = torch.zeros(pool, device="cuda")
    else:
        W, layer = case["W"], _layer(case)
        if kind == "load_refresh":
            s["ckpt"] = normal(1, n_slots, R, dv)
            s["states"] = torch.zeros(pool, device="cuda")
        else:                                            # a restored pool: omitted rows are zero
            s["states"] = normal(*pool)
            s["states"].view(n_slots, -1, dv)[:, s["inv_row"].long() < 0] = 0.0
        k = torch.randn((n, sh.n_qk_heads, W, sh.dk), generator=gen, device="cuda")
        s["k"] = (k / k.norm(dim=-1, keepdim=True)).to(torch.bfloat16)
        s["v"] = torch.randn((n, sh.n_heads, W, dv), generator=gen, device="cuda").to(torch.bfloat16)
        gs = (n, sh.n_heads, W, sh.dk) if sh.arch == "kda" else (n, sh.n_heads, W)
        rate = torch.as_tensor(lam[layer], dtype=torch.float32, device="cuda")
        rate = rate[None, :, None, :] if sh.arch == "kda" else rate[None, :, None]
        z = torch.randn(gs, generator=gen, device="cuda")
        s["g"] = (-rate * torch.nn.functional.softplus(z)).contiguous()
        s["beta"] = torch.sigmoid(torch.randn((n, sh.n_heads, W), generator=gen, device="cuda"))
        s["layer"], s["W"], s["init"] = layer, W, case["init"]
        ws = D.dasc_refresh_workspace_bytes(sh, n, W)    # kept between calls, as an engine does
        s["ws"] = torch.empty(ws, dtype=torch.uint8, device="cuda") if ws else None
    return s


def run(s):
    kind, sh = s["kind"], s["sh"]
    if kind == "pack":
        D.dasc_pack(sh, s["states"], s["src"], s["unit_row"], s["ckpt"], s["dst"], s["T"], s["C"])
        return s["ckpt"]
    if kind == "restore":
        D.dasc_restore(sh, s["ckpt"], s["src"], s["inv_row"], s["states"], s["dst"], s["n_rows"],
                       s["T"], s["C"])
        return s["states"]
    if kind == "pack_q8":
        D.dasc_pack_q8(sh, s["states"], s["src"], s["unit_row"], s["q"], s["scale"], s["dst"])
        return s["q"], s["scale"]
    if kind == "restore_q8":
        D.dasc_restore_q8(sh, s["q"], s["scale"], s["src"], s["inv_row"], s["states"], s["dst"], s["n_rows"])
        return s["states"]
    if kind == "refresh":
        D.dasc_refresh(sh, s["layer"], s["inv_row"], s["states"], s["dst"], s["k"], s["v"], s["g"],
                       s["beta"], s["W"], s["init"], workspace=s["ws"])
    else:
        D.dasc_restore_refresh(sh, s["layer"], s["ckpt"], s["src"], s["inv_row"], s["states"], s["dst"],
                               s["k"], s["v"], s["g"], s["beta"], s["W"], s["n_rows"],
                               init_mode=s["init"], workspace=s["ws"])
    return s["states"]


# ---- the work of one pass ------------------------------------------------------------------

def work(case):
    sh, p, _ = _plan_of(case)
    n, R, rows, dv, kind = case["n"], int(p["n_rows"]), sh.rows, sh.dv, case["kind"]
    row = 4 * dv
    if kind == "pack":
        return {"bytes": n * 2 * R * row, "flops": 0}
    if kind == "restore":
        return {"bytes": n * (R + rows) * row, "flops": 0}
    if kind == "pack_q8":
        return {"bytes": n * R * (row + dv + 4), "flops": 3 * n * R * dv}
    if kind == "restore_q8":
        return {"bytes": n * (R * (dv + 4) + rows * row), "flops": n * R * dv}
    # suffix inputs of the refreshed heads (k once per key head that one of them reads), the
    # state each starts from and the rows it writes; 5 operations per state entry and token
    lo, W, H = _layer(case) * sh.n_heads * sh.dk, case["W"], sh.n_heads
    omitted = p["inv_row"][lo:lo + H * sh.dk].reshape(H, sh.dk) < 0
    heads = np.flatnonzero(omitted.any(axis=1))
    keys = len(set(heads // (H // sh.n_qk_heads)))
    kept = int((~omitted).sum())
    b = keys * 2 * W * sh.dk + len(heads) * (2 * W * dv + 4 * W * (1 + (sh.dk if sh.arch == "kda" else 1)))
    if kind == "load_refresh":
        b += (kept + H * sh.dk) * row
    else:
        start = len(heads) * sh.dk * row if case["init"] == "restored" else 0
        b += start + int(omitted.sum()) * row
    return {"bytes": n * b, "flops": 5 * n * len(heads) * W * sh.dk * dv}


def tolerance(case):
    if "refresh" not in case["kind"]:
        return "exact"                       # copies, and codes that FP32 arithmetic fixes
    if case["dk"] == 128 and case["dv"] == 128:
        # products of split bf16 pairs, about 16 bits a term
        return {"rel": 3e-5}
    return {"rel": 2e-6}                     # fp32 per-token sums


# ---- the same in 64 bits ----------------------------------------------------------------

def _slots_of(packed, R):
    """[T, slots, C, dv] -> [slots, R, dv] (rank slices put end to end)."""
    return packed.permute(1, 0, 2, 3).reshape(packed.shape[1], -1, packed.shape[3])[:, :R]


def exact(case, seed):
    s = prepare(case, seed)
    sh, R, kind = s["sh"], s["n_rows"], s["kind"]
    src, dst = s["src"].long(), s["dst"].long()
    unit, inv = s["unit_row"].long(), s["inv_row"].long()
    dv = sh.dv
    if kind in ("pack", "restore"):
        return None                          # bit copies
    if kind == "pack_q8":
        scale = s["scale"].double()
        rows = s["states"].view(-1, sh.rows, dv)
        for a, b in zip(src.tolist(), dst.tolist()):
            scale[b] = rows[a, unit].abs().amax(dim=-1).double().clamp_min(1e-8) / 127.0
        return None, scale
    if kind == "restore_q8":
        out = s["states"].double().view(-1, sh.rows, dv)
        for a, b in zip(src.tolist(), dst.tolist()):
            out[b] = torch.where((inv >= 0)[:, None], s["q"][a, inv.clamp_min(0)].double()
                                 * s["scale"][a, inv.clamp_min(0)].double()[:, None], 0.0)
        return out.view(s["states"].shape)

    layer, H, dk, W = s["layer"], sh.n_heads, sh.dk, s["W"]
    inv_l = inv.view(sh.n_layers, H, dk)[layer]
    omitted = inv_l < 0
    out = s["states"].double()
    if kind == "load_refresh":
        packed = _slots_of(s["ckpt"], R)[src].double()
        S0 = torch.where(omitted[None, :, :, None], 0.0, packed[:, inv_l.clamp_min(0)])
    else:
        S0 = out[dst, layer]
    S = torch.zeros_like(S0) if s["init"] == "zero" else S0.clone()
    rep = H // sh.n_qk_heads
    for t in range(W):
        k = s["k"][:, :, t].double().repeat_interleave(rep, dim=1)          # [n, H, dk]
        g = s["g"][:, :, t].double()
        S.mul_(torch.exp(g)[..., None] if g.dim() == 3 else torch.exp(g)[..., None, None])
        y = (S * k[..., None]).sum(dim=2)                                   # S~^T k
        d = s["beta"][:, :, t].double()[..., None] * (s["v"][:, :, t].double() - y)
        S.addcmul_(k[..., None], d[:, :, None, :])
    out[dst, layer] = torch.where(omitted[None, :, :, None], S, S0)
    return out
