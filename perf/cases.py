"""The work that a user of this library has it do, as timed cases.

Each case is one call (or one cached step) through the public entry points of
`paper_2608_02474_amd.api` on seeded synthetic inputs made on the GPU: weights
N(0, 0.02), modulation shifts and scales N(0, 0.1) and gates N(0.25, 0.05),
latents N(0, 1) that drift by a per-frame amount from step to step, and frame
weights in [0, 1] of which some are those of silent frames (exact ties).

listed()          the cases
draw(rng)         one more case of the same ranges
prepare / run     a program's state before the call, and the call
work / tolerance  bytes and operations of a pass; how far outputs may differ
exact             the outputs in plain 64-bit torch
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_02474_amd import api

LN_EPS, XI, TAU = 1e-6, 1e-6, 0.9
_DT = {"bf16": torch.bfloat16, "f32": torch.float32}
_PI = math.pi


# ------------------------------------------------------------------- cases

def _case(name, kind, **kw):
    c = {"name": name, "kind": kind, "dtype": "bf16"}
    c.update(kw)
    return c


def listed() -> list:
    small = dict(T=5, gh=30, gw=52, D=1536, H=12, F=8960)      # 7800 tokens
    b480 = dict(T=21, gh=30, gw=52, D=5120, H=40, F=13824)     # 81 video frames at 480p: 32760 tokens
    b720 = dict(T=21, gh=45, gw=80, D=5120, H=40, F=13824)     # the same clip at 720p: 75600 tokens
    row480 = dict(T=21, gh=30, gw=52, D=5120)
    return [
        # the smallest whole step, all launches and no work: the fp32 exactness configuration
        _case("step_f32_32tok", "step", dtype="f32", T=2, gh=4, gw=4, D=64, H=2, F=256, K=16),
        # a small block with ragged tails in every tile size (the smoke configuration)
        _case("block_300tok", "block", T=3, gh=10, gw=10, D=256, H=2, F=512, K=111, invariant=False),
        # one block of the small configuration at its ratio of 0.25
        _case("block_7800tok", "block", K=1950, invariant=False, **small),
        # one scheduled step of a four-block model of that size: selection, K from the schedule, every block
        _case("stack_7800tok", "stack", blocks=4, **small),
        # the block with qk norm, 3D rotary and cross-attention, batch of two for guidance
        _case("wan_7800tok_b2", "wan", B=2, Lc=512, K=1950, invariant=False, **small),
        # a late denoising step at 480p: little changed, a tenth of the tokens recomputed
        _case("block_480p_k3276", "block", K=3276, invariant=False, **b480),
        # the headline: a whole cached step of the 14B-shaped block at 480p
        _case("step_480p_k13104", "step", K=13104, **b480),
        # the largest block: the same clip at 720p
        _case("block_720p_k22680", "block", K=22680, invariant=False, **b720),
        # the saliency and selection alone, as a program that picks its own blocks calls them
        _case("select_480p", "select", mode="topk", K=13104, **row480),
        # the cache write and fusion alone, int8 residual codec
        _case("cache_480p", "cache", codec=0, K=13104, **row480),
        # one update of the adaptive reference cache, chains of one latent-grid row
        _case("refcache_480p", "refcache", K=13104, **row480),
        # the audio anchor of a clip of 81 frames at 16 per second
        _case("energy_81000", "energy", T=21, n_samples=81000, n_fft=512, hop=160, n_bands=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, lo, hi):
    """T, gh, gw with about a log-uniform number of tokens in [lo, hi]."""
    while True:
        n = _log_int(rng, lo, hi)
        T = rng.randint(1, 21)
        gh = max(1, int(round(math.sqrt(n / T / rng.uniform(1.0, 2.0)))))
        gw = max(1, int(round(n / T / gh)))
        if lo <= T * gh * gw <= hi:
            return dict(T=T, gh=gh, gw=gw)


def draw(rng) -> dict:
    """One more case: the same kinds, sizes spread over the whole range."""
    limit = _block_flops(75600, 22680, 5120, 13824)
    while True:
        kind = rng.choice(["block", "block", "step", "stack", "wan", "select", "cache", "refcache", "energy", "step_f32"])
        if kind == "energy":
            return {"kind": kind, "dtype": "bf16", "T": rng.randint(1, 40), "n_samples": _log_int(rng, 4000, 480000),
                    "n_fft": rng.choice([256, 400, 512, 512, 1024]), "hop": rng.choice([128, 160, 160, 256]),
                    "n_bands": rng.choice([4, 8, 8, 16])}
        if kind == "step_f32":
            dh = rng.choice([16, 32, 64, 128])
            H = rng.randint(1, 4)
            c = {"kind": "step", "dtype": "f32", **_grid(rng, 16, 600), "D": dh * H, "H": H,
                 "F": 8 * rng.randint(8, 128)}
            c["K"] = rng.randint(1, _tokens(c))
            return c
        if kind in ("select", "cache", "refcache"):
            c = {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "bf16", "f32"]), **_grid(rng, 200, 75600),
                 "D": 8 * _log_int(rng, 32, 640)}
            if _tokens(c) * c["D"] > 75600 * 5120 // (2 if c["dtype"] == "f32" else 1):
                continue
            c["K"] = max(1, int(rng.uniform(0.05, 1.0) * _tokens(c)))
            if kind == "select":
                c["mode"] = rng.choice(["topk", "topk", "threshold", "two_stage"])
            if kind == "cache":
                c["codec"] = rng.choice([0, 0, 1, 2])
            return c
        D = 256 * _log_int(rng, 1, 20)
        c = {"kind": kind, "dtype": "bf16", **_grid(rng, 200, 75600), "D": D, "H": D // 128,
             "F": 256 * max(1, int(round(D * rng.uniform(2.0, 6.0) / 256)))}
        L = _tokens(c)
        c["K"] = max(1, int(rng.uniform(0.05, 1.0) * L))
        if kind == "stack":
            del c["K"]
            c["blocks"] = rng.randint(2, 4)
            if _block_flops(L, L, D, c["F"]) * c["blocks"] > limit / 4:
                continue
        elif kind == "wan":
            c["B"], c["Lc"], c["invariant"] = rng.randint(1, 2), _log_int(rng, 16, 600), rng.random() < 0.1
            if c["B"] * _block_flops(L, c["K"], D, c["F"]) > limit / 2:
                continue
        else:
            if kind == "block":
                c["invariant"] = rng.random() < 0.1
            if _block_flops(L, c["K"], D, c["F"]) > limit * 0.9:
                continue
        return c


def _tokens(c) -> int:
    return c["T"] * c["gh"] * c["gw"]


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1 + 1000003 * int(seed))
    return g


def _randn(g, *shape, std=1.0, dt=torch.float32):
    return torch.randn(shape, device="cuda", generator=g).mul_(std).to(dt)


def _weights(c, g, wan=False) -> dict:
    D, F, dt = c["D"], c["F"], _DT[c["dtype"]]
    p = {n: _randn(g, *s, std=0.02, dt=dt) for n, s in
         (("wq", (D, D)), ("wk", (D, D)), ("wv", (D, D)), ("wo", (D, D)), ("w1", (F, D)), ("w2", (D, F)),
          ("bq", (D,)), ("bk", (D,)), ("bv", (D,)), ("bo", (D,)), ("b1", (F,)), ("b2", (D,)))}
    mod = _randn(g, 6, D, std=0.1)
    for r in (2, 5):
        mod[r] = 0.25 + 0.05 * torch.randn(D, device="cuda", generator=g)
    p["mod"] = mod
    if wan:
        for n in ("wqc", "wkc", "wvc", "woc"):
            p[n] = _randn(g, D, D, std=0.02, dt=dt)
        for n in ("bqc", "bkc", "bvc", "boc"):
            p[n] = _randn(g, D, std=0.02, dt=dt)
        for n in ("gq", "gk", "gqc", "gkc", "g3"):
            p[n] = 1.0 + 0.1 * torch.randn(D, device="cuda", generator=g)
        p["b3"] = _randn(g, D, std=0.02)
    return p


def _frame_weight(c, g):
    fw = torch.rand(c["T"], device="cuda", generator=g)
    fw[torch.rand(c["T"], device="cuda", generator=g) < 0.15] = 0.0     # silent frames
    return fw


def _drift(x, c, g):
    """The next step's latents: every frame moves by an amount of its own."""
    sig = 0.01 + 0.29 * torch.rand(c["T"], device="cuda", generator=g)
    n = torch.randn(x.shape, device="cuda", generator=g)
    n.mul_(sig.repeat_interleave(c["gh"] * c["gw"])[:, None]).add_(x)
    return n.to(x.dtype)


def _selection(L, K, g):
    mask = torch.zeros(L, dtype=torch.uint8, device="cuda")
    idx = torch.randperm(L, device="cuda", generator=g)[:K].sort().values.to(torch.int32)
    mask[idx.long()] = 1
    return idx, mask


def _audio(c, seed):
    """Harmonic bursts with pauses at 16 kHz."""
    r = np.random.default_rng(int(seed))
    n, sr, pos = c["n_samples"], 16000, 0
    out = np.zeros(n, np.float32)
    while pos < n:
        m = min(int(r.uniform(0.15, 0.5) * sr), n - pos)
        t = np.arange(m) / sr
        f0 = r.uniform(90.0, 250.0)
        s = sum(np.cos(2 * np.pi * h * f0 * t + r.uniform(0, 6.28)) / h for h in range(1, 7))
        out[pos:pos + m] = s * r.uniform(0.05, 0.3)
        pos += m + int(r.uniform(0.05, 0.35) * sr)
    return torch.from_numpy(out).cuda()


def _chain_outputs(c, g):
    """Fresh outputs that are alike along a chain (one latent-grid row): a
    shared part, and an AR(1) sequence along the row."""
    n, w, D = c["T"] * c["gh"], c["gw"], c["D"]
    y = torch.randn((n, w, D), device="cuda", generator=g)
    for t in range(1, w):
        y[:, t].mul_((1.0 - 0.95 ** 2) ** 0.5).add_(y[:, t - 1], alpha=0.95)
    y += 2.0 * torch.randn((n, 1, D), device="cuda", generator=g)
    return y.reshape(n * w, D)


def _inputs(case, seed) -> dict:
    """What prepare() and exact() both start from."""
    c, g = case, _gen(seed)
    if c["kind"] == "energy":
        return {"audio": _audio(c, seed)}
    L, D, dt, kind = _tokens(c), c["D"], _DT[c["dtype"]], c["kind"]
    s = {}
    if kind == "block":
        s["p"] = _weights(c, g)
        s["x"] = _randn(g, L, D, dt=dt)
        s["idx"], _ = _selection(L, c["K"], g)
    elif kind == "wan":
        s["p"] = _weights(c, g, wan=True)
        s["x"] = _randn(g, c["B"], L, D, dt=dt)
        s["ctx"] = _randn(g, c["B"], c["Lc"], D, dt=dt)
        s["idx"] = torch.cat([b * L + _selection(L, c["K"], g)[0] for b in range(c["B"])]).to(torch.int32)
    elif kind == "step":
        s["p"] = _weights(c, g)
        s["fw"] = _frame_weight(c, g)
        s["x0"] = _randn(g, L, D, dt=dt)
        s["y0"] = s["x0"].float() + 0.3 * torch.randn((L, D), device="cuda", generator=g)
        s["xs"] = [_drift(s["x0"], c, g) for _ in range(2)]
    elif kind == "stack":
        s["ps"] = [_weights(c, g) for _ in range(c["blocks"])]
        s["fw"] = _frame_weight(c, g)
        s["x0"] = _randn(g, L, D, dt=dt)
        s["xs"] = [_drift(s["x0"], c, g) for _ in range(2)]
    elif kind == "select":
        s["xref"] = _randn(g, L, D, dt=dt)
        s["x"] = _drift(s["xref"], c, g)
        s["fw"] = _frame_weight(c, g)
        s["keys"] = torch.rand(c["T"], device="cuda", generator=g)
    elif kind == "cache":
        s["x0"] = _randn(g, L, D, dt=dt)
        s["y0"] = s["x0"].float() + 0.3 * torch.randn((L, D), device="cuda", generator=g)
        s["x"] = _drift(s["x0"], c, g)
        s["idx"], s["mask"] = _selection(L, c["K"], g)
        s["y_sel"] = s["x"][s["idx"].long()].float() + 0.3 * torch.randn((c["K"], D), device="cuda", generator=g)
    elif kind == "refcache":
        s["x"] = _randn(g, L, D, dt=dt)
        s["y0"] = _chain_outputs(c, g)
        s["sels"] = []
        for _ in range(2):
            idx, mask = _selection(L, c["K"], g)
            y = s["y0"][idx.long()] + 0.05 * torch.randn((c["K"], D), device="cuda", generator=g)
            s["sels"].append((idx, mask, y))
    else:
        raise ValueError(kind)
    return s


# --------------------------------------------------------- prepare and run

def prepare(case, seed) -> dict:
    c, s = case, _inputs(case, seed)
    s["c"], s["at"], s["ws"] = c, 0, api.Workspace()
    kind = c["kind"]
    if kind == "energy":
        return s
    L, D, dt = _tokens(c), c["D"], _DT[c["dtype"]]
    every = torch.arange(L, dtype=torch.int32, device="cuda")
    ones = torch.ones(L, dtype=torch.uint8, device="cuda")
    if kind == "block":
        s["y_sel"] = torch.empty((c["K"], D), dtype=torch.float32, device="cuda")
    elif kind == "wan":
        s["y_sel"] = torch.empty((c["B"] * c["K"], D), dtype=torch.float32, device="cuda")
    elif kind == "step":
        # a block whose cache was filled by the step before
        s["blk"] = blk = api.CachedBlock(s["p"], c["H"], L, D, "cuda", dt, LN_EPS, XI)
        api.cache_update(s["x0"], every, ones, L, s["y0"], blk.xref, blk.codes, blk.scale, blk.y)
        del s["x0"], s["y0"]
    elif kind == "stack":
        # after its first, full step
        s["stack"] = api.BlockStack(s["ps"], c["H"], L, D, torch.device("cuda"), dt,
                                    api.Scheduler(1, 0.2, 0.6, 0.4), XI, LN_EPS)
        s["stack"].step(s["x0"], s["fw"], c["gh"] * c["gw"])
    elif kind == "cache":
        s["xref"] = torch.zeros((L, D), dtype=dt, device="cuda")
        s["store"] = torch.zeros((L, D), dtype=dt, device="cuda") if c["codec"] == 1 else None
        s["codes"] = torch.zeros((L, D), dtype=torch.int8, device="cuda") if c["codec"] != 1 else None
        s["scale"] = torch.zeros(L, dtype=torch.float32, device="cuda") if c["codec"] != 1 else None
        s["y"] = torch.empty((L, D), dtype=dt, device="cuda")
        api.cache_update_codec(c["codec"], s["x0"], every, ones, L, s["y0"], s["xref"], s["y"], s["store"],
                               s["codes"], s["scale"])
        del s["x0"], s["y0"]
    elif kind == "refcache":
        s["rc"] = rc = api.RefCache(L, D, c["gw"], TAU, dt, "cuda")
        rc.codes.zero_()        # a reference entry has no codes of its own
        s["xref"] = torch.zeros((L, D), dtype=dt, device="cuda")
        s["y"] = torch.empty((L, D), dtype=dt, device="cuda")
        rc.update(s["x"], every, ones, L, s["y0"], s["xref"], s["y"])
        del s["y0"]
    return s


def run(s):
    c = s["c"]
    kind = c["kind"]
    if kind == "block":
        return api.block_partial(s["p"], s["x"], s["idx"], c["K"], c["H"], LN_EPS, y_sel=s["y_sel"],
                                 workspace=s["ws"], batch_invariant=c["invariant"])
    if kind == "wan":
        return api.wan_block_partial(s["p"], s["x"], s["ctx"], s["idx"], [c["K"]] * c["B"], c["H"],
                                     (c["T"], c["gh"], c["gw"]), y_sel=s["y_sel"], workspace=s["ws"],
                                     batch_invariant=c["invariant"])
    if kind == "energy":
        return api.energy(s["audio"], c["T"], 16000, c["n_fft"], c["hop"], c["n_bands"], workspace=s["ws"])
    N = c["gh"] * c["gw"]
    if kind == "step":
        blk = s["blk"]
        x = s["xs"][s["at"] % 2]        # the trajectory's next latents
        s["at"] += 1
        y = blk.step(x, s["fw"], N, k=c["K"])
        return {"y": y, "y_sel": blk.y_sel[:c["K"]], "idx": blk.sel.idx[:c["K"]], "mask": blk.sel.mask,
                "saliency": blk.sel.saliency, "step_delta": blk.sel.step_delta, "xref": blk.xref,
                "scale": blk.scale}
    if kind == "stack":
        x = s["xs"][s["at"] % 2]
        s["at"] += 1
        st = s["stack"]
        y = st.step(x, s["fw"], N)
        return {"y": y, "K": st.history[-1][0], "delta": st.history[-1][2], "xref": list(st.xref),
                "scale": list(st.scale)}
    if kind == "select":
        if c["mode"] == "two_stage":
            n = max(1, 2 * c["T"] // 3)
            k = max(1, c["K"] // n)
            sel = api.saliency(s["x"], s["xref"], s["fw"], N, XI, workspace=s["ws"])
            sel = api.topk_segments(sel, api.anchors(c["T"], n, "energy", s["keys"]), N, k)
            count = api.segments_count(n, N, k)
        elif c["mode"] == "threshold":
            sel = api.select(s["x"], s["xref"], s["fw"], N, threshold=0.05, xi=XI, workspace=s["ws"])
            return {"mask": sel.mask, "n": sel.n_sel_dev, "saliency": sel.saliency, "step_delta": sel.step_delta}
        else:
            sel = api.select(s["x"], s["xref"], s["fw"], N, k=c["K"], xi=XI, workspace=s["ws"])
            count = c["K"]
        return {"idx": sel.idx[:count], "mask": sel.mask, "n": sel.n_sel_dev, "saliency": sel.saliency,
                "step_delta": sel.step_delta}
    if kind == "cache":
        y = api.cache_update_codec(c["codec"], s["x"], s["idx"], s["mask"], c["K"], s["y_sel"], s["xref"], s["y"],
                                   s["store"], s["codes"], s["scale"])
        out = {"y": y, "xref": s["xref"]}
        out.update({"store": s["store"]} if c["codec"] == 1 else {"codes": s["codes"], "scale": s["scale"]})
        return out
    idx, mask, y_sel = s["sels"][s["at"] % 2]
    s["at"] += 1
    rc = s["rc"]
    y = rc.update(s["x"], idx, mask, c["K"], y_sel, s["xref"], s["y"])
    return {"y": y, "kind": rc.ent_kind, "codes": rc.codes, "scale": rc.scale, "xref": s["xref"],
            "free": rc.free_top[:1]}


# -------------------------------------------------------- work, tolerances

def _block_flops(L, K, D, F):
    return 4 * L * D * D + 4 * K * D * D + 4 * K * L * D + 4 * K * D * F


def work(case) -> dict:
    c, kind = case, case["kind"]
    if kind == "energy":
        m = c["n_samples"] // c["T"]
        frames = c["T"] * (1 if m < c["n_fft"] else 1 + (m - c["n_fft"]) // c["hop"])
        return {"bytes": 4 * c["n_samples"] + 4 * c["T"] * (2 + c["n_bands"]),
                "flops": int(frames * 2.5 * c["n_fft"] * math.log2(c["n_fft"]))}
    L, D, b = _tokens(c), c["D"], 2 if c["dtype"] == "bf16" else 4
    if kind == "select":
        return {"bytes": 2 * L * D * b + 9 * L, "flops": 4 * L * D}
    if kind in ("cache", "refcache"):
        K, U = c["K"], L - c["K"]
        # fresh rows: y_sel and x read, y, the reference and the entry written; reused rows: entry read, y written
        fresh = {0: 3 * b + 1, 1: 4 * b, 2: 3 * b + 1}[c.get("codec", 0)]
        reuse = {0: 2 * b + 1, 1: 2 * b, 2: b + 1}[c.get("codec", 0)]
        return {"bytes": K * D * (4 + fresh) + U * D * reuse + 5 * L, "flops": 6 * L * D}
    F = c["F"]
    wb = (4 * D * D + 2 * D * F) * b
    if kind == "block":
        return {"bytes": L * D * b + wb + 4 * c["K"] * D + 4 * c["K"], "flops": _block_flops(L, c["K"], D, F)}
    if kind == "wan":
        B, K, Lc = c["B"], c["K"], c["Lc"]
        cross = 4 * K * D * D + 4 * Lc * D * D + 4 * K * Lc * D
        return {"bytes": B * (L + Lc) * D * b + wb + 4 * D * D * b + 4 * B * K * D,
                "flops": B * (_block_flops(L, K, D, F) + cross)}
    if kind == "step":
        K = c["K"]
        return {"bytes": L * D * (3 * b + 1) + K * D * b + wb + 4 * K * D, "flops": _block_flops(L, K, D, F)}
    K, n = int(0.5 * L), c["blocks"]          # the schedule's K lies in [0.2 L, 0.6 L]
    return {"bytes": L * D * b + n * (wb + L * D * (b + 1) + K * D * b), "flops": n * _block_flops(L, K, D, F)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("cache", "refcache"):
        return "exact"          # the codes, scales and rows are defined bit by bit in fp32
    # about four times the error against exact() that the calls show
    if kind in ("select", "energy"):
        return {"rel": 2e-7, "max": 2e-6, "differ": 1e-4}    # fp64 sums rounded once; ties at the threshold
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 2e-5}
    if kind == "stack":
        return {"rel": 1.5e-2, "max": 0.3}      # a rounding of one block travels through those after it
    if kind == "step":
        return {"rel": 6e-3, "max": 0.1}        # bf16 rows, reused ones among them
    return {"rel": min(5e-3, 1.5e-6 * case["D"]), "max": 0.1}   # D = 256: 4.8e-5, 1536: 5.6e-4, 5120: 1.2e-3


# ------------------------------------------------------------------- exact

def _ln(z):
    m = z.mean(1, keepdim=True)
    d = z - m
    return d / torch.sqrt((d * d).mean(1, keepdim=True) + LN_EPS)


def _attend(q, k, v, H):
    dh = q.shape[1] // H
    o = torch.empty_like(q)
    for h in range(H):
        a = slice(h * dh, (h + 1) * dh)
        kt, vh = k[:, a].t().contiguous(), v[:, a].contiguous()
        for r in range(0, q.shape[0], 8192):
            o[r:r + 8192, a] = torch.softmax(q[r:r + 8192, a].contiguous() @ kt / math.sqrt(dh), dim=1) @ vh
    return o


def _gelu(z):
    return 0.5 * z * (1.0 + torch.tanh(math.sqrt(2.0 / _PI) * (z + 0.044715 * z ** 3)))


def _lin(a, p, w, b):
    return torch.addmm(p[b].double(), a, p[w].double().t())


def _block64(p, x, idx, H):
    """The block's fp64 output rows idx of the inputs x."""
    m = p["mod"].double()
    xd = x.double()
    a = _ln(xd) * (1.0 + m[1]) + m[0]
    i = idx.long()
    o = _attend(_lin(a[i], p, "wq", "bq"), _lin(a, p, "wk", "bk"), _lin(a, p, "wv", "bv"), H)
    x1 = xd[i] + m[2] * _lin(o, p, "wo", "bo")
    h = _gelu(_lin(_ln(x1) * (1.0 + m[4]) + m[3], p, "w1", "b1"))
    return x1 + m[5] * _lin(h, p, "w2", "b2")


def _rms(z, g):
    return z / torch.sqrt((z * z).mean(1, keepdim=True) + 1e-6) * g.double()


def _rope(z, pos, c):
    dh = z.shape[1] // c["H"]
    n3 = dh // 6
    nt = dh // 2 - 2 * n3
    gh, gw = c["gh"], c["gw"]
    at = (pos // (gh * gw), (pos // gw) % gh, pos % gw)
    ang = torch.cat([p.double()[:, None] * 10000.0 ** (-torch.arange(n, device="cuda", dtype=torch.float64) / n)
                     for p, n in zip(at, (nt, n3, n3))], dim=1)[:, None, :]
    v = z.reshape(z.shape[0], c["H"], dh // 2, 2)
    a, b = v[..., 0], v[..., 1]
    return torch.stack([a * ang.cos() - b * ang.sin(), a * ang.sin() + b * ang.cos()], dim=-1).reshape(z.shape)


def _wan64(p, x, ctx, i, c):
    m = p["mod"].double()
    xd, pos = x.double(), torch.arange(x.shape[0], device="cuda")
    a = _ln(xd) * (1.0 + m[1]) + m[0]
    q = _rope(_rms(_lin(a[i], p, "wq", "bq"), p["gq"]), i, c)
    k = _rope(_rms(_lin(a, p, "wk", "bk"), p["gk"]), pos, c)
    x1 = xd[i] + m[2] * _lin(_attend(q, k, _lin(a, p, "wv", "bv"), c["H"]), p, "wo", "bo")
    n = _ln(x1) * p["g3"].double() + p["b3"].double()
    q = _rms(_lin(n, p, "wqc", "bqc"), p["gqc"])
    cd = ctx.double()
    k = _rms(_lin(cd, p, "wkc", "bkc"), p["gkc"])
    x2 = x1 + _lin(_attend(q, k, _lin(cd, p, "wvc", "bvc"), c["H"]), p, "woc", "boc")
    h = _gelu(_lin(_ln(x2) * (1.0 + m[4]) + m[3], p, "w1", "b1"))
    return x2 + m[5] * _lin(h, p, "w2", "b2")


def _saliency64(x, xref, fw, N):
    """(s rounded once to fp32, the step's value)"""
    num, den = [], []
    for r in range(0, x.shape[0], 8192):
        a, b = x[r:r + 8192].double(), xref[r:r + 8192].double()
        num.append((a - b).abs().sum(1))
        den.append(b.abs().sum(1))
    num, den = torch.cat(num), torch.cat(den)
    s = (fw.double().repeat_interleave(N) * (num / (den + XI))).float()
    return s, (num.sum() / (den.sum() + XI)).reshape(1)


def _topk(s, k):
    idx = torch.sort(s, descending=True, stable=True).indices[:k].sort().values.to(torch.int32)
    mask = torch.zeros(s.numel(), dtype=torch.uint8, device="cuda")
    mask[idx.long()] = 1
    return idx, mask


def _quantize(src):
    """Codes and scales of fp32 rows (the code is an integer that fp32 arithmetic decides)."""
    amax = src.abs().amax(1, keepdim=True)
    nz = amax > 0
    inv = torch.where(nz, 127.0 / amax, torch.zeros_like(amax))
    scale = torch.where(nz, amax / 127.0, torch.zeros_like(amax))
    return torch.clamp(torch.round(src * inv), -127, 127).to(torch.int8), scale[:, 0].contiguous()


def _dequantize(ref, scale, codes):
    return scale.double()[:, None] * codes.double() + (0.0 if ref is None else ref.double())


def exact(case, seed):
    c, s, kind = case, _inputs(case, seed), case["kind"]
    if kind == "energy":
        a, T, n = s["audio"].double().cpu(), c["T"], c["n_fft"]
        win = 0.5 - 0.5 * torch.cos(2 * _PI * torch.arange(n, dtype=torch.float64) / n)
        f = torch.arange(n // 2 + 1, dtype=torch.float64) * 16000 / n
        mel = lambda v: 2595.0 * torch.log10(1.0 + v / 700.0)  # noqa: E731
        top = mel(torch.tensor(8000.0, dtype=torch.float64)) / c["n_bands"]
        band = torch.clamp(torch.floor(mel(f) / top), max=c["n_bands"] - 1).long()
        out = torch.zeros((T, c["n_bands"]), dtype=torch.float64)
        for t in range(T):
            seg = a[t * a.numel() // T:(t + 1) * a.numel() // T]
            if seg.numel() < n:
                seg = torch.cat([seg, torch.zeros(n - seg.numel(), dtype=torch.float64)])
            pw = torch.fft.rfft(seg.unfold(0, n, c["hop"]) * win).abs().square().sum(0)
            out[t].index_add_(0, band, pw)
        e = out.sum(1).sqrt()
        return [out, e, e / e.max() if e.max() > 0 else torch.ones_like(e)]
    L, N = _tokens(c), c["gh"] * c["gw"]
    if kind == "block":
        return _block64(s["p"], s["x"], s["idx"], c["H"])
    if kind == "wan":
        K = c["K"]
        return torch.cat([_wan64(s["p"], s["x"][b], s["ctx"][b], s["idx"][b * K:(b + 1) * K].long() - b * L, c)
                          for b in range(c["B"])])
    if kind == "step":
        x = s["xs"][0]
        sal, delta = _saliency64(x, s["x0"], s["fw"], N)
        idx, mask = _topk(sal, c["K"])
        i = idx.long()
        ys = _block64(s["p"], x, idx, c["H"])
        codes, scale = _quantize(s["y0"] - s["x0"].float())
        y = _dequantize(s["x0"], scale, codes)
        y[i] = ys
        xref = s["x0"].clone()
        xref[i] = x[i]
        scale[i] = _quantize(ys.float() - x[i].float())[1]
        return {"y": y, "y_sel": ys, "idx": idx, "mask": mask, "saliency": sal.double(), "step_delta": delta,
                "xref": xref.double(), "scale": scale.double()}
    if kind == "stack":
        x, refs, codes, scales = s["x0"].double(), [], [], []
        for p in s["ps"]:
            ys = _block64(p, x, torch.arange(L, device="cuda"), c["H"])
            q, sc = _quantize((ys - x).float())
            refs.append(x), codes.append(q), scales.append(sc)
            x = ys
        sal, delta = _saliency64(s["xs"][0], s["x0"], s["fw"], N)
        K = int(math.ceil(0.6 * L - 1e-9))      # the first cached step: its delta is the largest so far
        i = _topk(sal, K)[0].long()
        x = s["xs"][0].double()
        for b, p in enumerate(s["ps"]):
            ys = _block64(p, x, i, c["H"])
            y = _dequantize(refs[b], scales[b], codes[b])
            y[i] = ys
            refs[b][i] = x[i]
            scales[b][i] = _quantize((ys - x[i]).float())[1]
            x = y
        return {"y": x, "K": None, "delta": float(delta), "xref": refs, "scale": [v.double() for v in scales]}
    if kind == "select":
        sal, delta = _saliency64(s["x"], s["xref"], s["fw"], N)
        out = {"saliency": sal.double(), "step_delta": delta}
        if c["mode"] == "topk":
            out["idx"], out["mask"] = _topk(sal, c["K"])
        return out
    if kind == "cache":
        x, i, ys = s["x"], s["idx"].long(), s["y_sel"]
        xref = s["x0"].clone()
        dt = x.dtype
        if c["codec"] == 1:
            y = s["y0"].to(dt)
            y[i] = ys.to(dt)
            xref[i] = x[i]
            return {"y": y.double(), "xref": xref.double(), "store": y.double()}
        codes, scale = _quantize(s["y0"] - s["x0"].float() if c["codec"] == 0 else s["y0"])
        y = _dequantize(s["x0"] if c["codec"] == 0 else None, scale, codes)
        y[i] = ys.double()
        codes[i], scale[i] = _quantize(ys - x[i].float() if c["codec"] == 0 else ys)
        xref[i] = x[i]
        return {"y": y, "xref": xref.double(), "codes": codes, "scale": scale.double()}
    return _refcache64(c, s)


def _refcache64(c, s):
    n, w, D, dt = c["T"] * c["gh"], c["gw"], c["D"], _DT[c["dtype"]]
    L = n * w
    ref = torch.zeros((n, D), dtype=dt, device="cuda")          # each chain's current reference
    have = torch.zeros(n, dtype=torch.bool, device="cuda")
    entry = torch.zeros((n, w, D), dtype=dt, device="cuda")     # the reference behind each token
    codes = torch.zeros((n, w, D), dtype=torch.int8, device="cuda")
    scale = torch.zeros((n, w), dtype=torch.float32, device="cuda")
    kind = torch.zeros((n, w), dtype=torch.uint8, device="cuda")

    def write(y, mask):
        nonlocal ref
        for t in range(w):
            m = mask[:, t]
            v = y[:, t]
            rd, vd = ref.double(), v.double()
            yy, rr = (vd * vd).sum(1), (rd * rd).sum(1)
            sim = torch.where((yy == 0) | (rr == 0), torch.zeros_like(yy), (vd * rd).sum(1) / (yy.sqrt() * rr.sqrt()))
            res = m & have & (sim > float(np.float32(TAU)))
            new = m & ~res
            ref = torch.where(new[:, None], v.to(dt), ref)
            have.logical_or_(new)
            q, sc = _quantize(v - ref.float())
            codes[:, t] = torch.where(res[:, None], q, codes[:, t])
            scale[:, t] = torch.where(res, sc, torch.where(new, torch.zeros_like(sc), scale[:, t]))
            entry[:, t] = torch.where(m[:, None], ref, entry[:, t])
            kind[:, t] = torch.where(res, 2, torch.where(new, 1, kind[:, t].long())).to(torch.uint8)

    write(s["y0"].reshape(n, w, D), torch.ones((n, w), dtype=torch.bool, device="cuda"))
    idx, mask, ys = s["sels"][0]
    i = idx.long()
    full = torch.zeros((L, D), dtype=torch.float32, device="cuda")
    full[i] = ys
    write(full.reshape(n, w, D), mask.bool().reshape(n, w))
    q = torch.where((kind == 2)[..., None], codes, torch.zeros_like(codes)).reshape(L, D)
    y = _dequantize(entry.reshape(L, D), scale.reshape(L), q)
    y[i] = ys.double()
    return {"y": y, "kind": kind.reshape(L), "codes": codes.reshape(L, D), "scale": scale.reshape(L).double(),
            "xref": s["x"].double(), "free": None}
